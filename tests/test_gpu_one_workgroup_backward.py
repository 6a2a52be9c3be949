"""Backward calls of a few token groups, which one workgroup computes in full (dalpha and dbeta written by
the kernel itself), and the first sizes beyond, which go through partial rows: every output against the
oracle, the outputs of partial calls bit for bit those of the full one, and the bytes after dalpha and
dbeta untouched."""
import pytest
import torch

import oracle
import paper_2603_08343_amd as wht
from paper_2603_08343_amd import synth
from parity import assert_grad_close, assert_io_close, to_gpu

pytestmark = pytest.mark.gpu

# width, dtype, tokens of a workgroup pass
SHAPES = [(32, "bf16", 64), (512, "bf16", 8), (768, "bf16", 8), (1024, "bf16", 4), (1536, "bf16", 4), (2048, "bf16", 4),
          (3072, "bf16", 2), (4096, "bf16", 2), (6144, "bf16", 1), (8192, "bf16", 1), (12288, "bf16", 1),
          (16384, "bf16", 1), (64, "f32", 32), (1024, "f32", 4), (2048, "f32", 4), (4096, "f32", 1), (8192, "f32", 1)]


@pytest.mark.parametrize("d,dtype,G", SHAPES)
def test_few_groups(d, dtype, G):
    # 768: four tokens to a workgroup up to 4 and from 17 to 512
    more = {4, 5, 511, 512, 513} if d == 768 else set()
    for N in sorted({1, G, G + 1, 2 * G, 2 * G + 1, 3 * G, 3 * G + 1} | more):
        print(f"[one workgroup] d={d} {dtype} N={N}", flush=True)
        inp = synth.make_inputs(N, d, dtype, seed=11 * d + N)
        x, dy = to_gpu(inp.x, dtype), to_gpu(inp.dy, dtype)
        a = torch.from_numpy(inp.alpha).cuda()
        fence = torch.full((2, d + 64), 5.0, device="cuda")
        dx, da, db = wht.wht_affine_backward(dy, x, a, dalpha=fence[0, :d], dbeta=fence[1, :d])
        _, da1, db1 = wht.wht_affine_backward(dy, x, a, want_dx=False)
        dx1 = wht.wht_affine_backward(dy, None, a, want_param_grads=False)[0]
        torch.cuda.synchronize()
        rdx, rda, rdb = oracle.backward(inp.dy, inp.x, inp.alpha, "fast")
        assert_io_close(dx, rdx, dtype, f"dx d={d} N={N}")
        assert_grad_close(da, rda, f"dalpha d={d} N={N}")
        assert_grad_close(db, rdb, f"dbeta d={d} N={N}")
        assert torch.equal(da, da1) and torch.equal(db, db1) and torch.equal(dx, dx1)
        assert bool((fence[:, d:] == 5.0).all())
