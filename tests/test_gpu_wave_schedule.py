"""The wave schedule (every stage in registers or between lanes; float32 tensors, and bfloat16 below
d = 1024) where it can go wrong: token counts around a workgroup pass (a wave holds 64 * values-per-lane
/ d tokens), one token, and the size at which the forward call changes from the one-pass to the
persistent kernel.  Tolerances as in parity.py; the two forward kernels do the same arithmetic in the
same order, so their results have to be equal bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_08343_amd as wht
import routes
from paper_2603_08343_amd import synth
from parity import assert_grad_close, assert_io_close, nan_filled, to_gpu

pytestmark = pytest.mark.gpu

F32 = [(1 << n, "f32") for n in range(5, 14)]
BF16 = [(1 << n, "bf16") for n in range(5, 10)]


def _tokens_per_pass(d, dtype):
    """256 threads of 16 values (an eighth of a short row, 32 where 64 lanes of 16 would not hold the row);
    one token where it takes two or four waves.  The library's rule, restated."""
    per_lane = min(16, max(d // 8, 4 if dtype == "f32" else 8))
    if d > 64 * per_lane:
        per_lane = 32
    return 256 * per_lane // d if d <= 64 * per_lane else 1


@pytest.mark.parametrize("d,dtype", F32 + BF16)
def test_backward_around_a_workgroup_pass(d, dtype):
    G = _tokens_per_pass(d, dtype)
    for N in sorted({1, max(1, G // 4 - 1), max(1, G - 1), G, G + 1, 3 * G + max(1, G // 4) + 1}):
        print(f"[wave] backward d={d} {dtype} N={N}", flush=True)
        inp = synth.make_inputs(N, d, dtype, seed=7 * d + N)
        x, dy = to_gpu(inp.x, dtype), to_gpu(inp.dy, dtype)
        a = torch.from_numpy(inp.alpha).cuda()
        buf = nan_filled(N + 1, d, dtype)                    # the row after the last must keep its fill
        dx, da, db = wht.wht_affine_backward(dy, x, a, dx=buf[:N])
        torch.cuda.synchronize()
        rdx, rda, rdb = oracle.backward(inp.dy, inp.x, inp.alpha, "fast")
        assert_io_close(dx, rdx, dtype, f"dx d={d} N={N}")
        assert_grad_close(da, rda, f"dalpha d={d} N={N}")
        assert_grad_close(db, rdb, f"dbeta d={d} N={N}")
        assert bool(torch.isnan(buf[N].float()).all())


@pytest.mark.parametrize("N", [257, 768, 769])
def test_backward_where_the_grid_changes(N):
    # float32 d = 4096: one workgroup per CU up to 768 tokens, two beyond
    d = 4096
    print(f"[wave] backward d={d} f32 N={N}", flush=True)
    inp = synth.make_inputs(N, d, "f32", seed=N)
    x, dy = to_gpu(inp.x, "f32"), to_gpu(inp.dy, "f32")
    dx, da, db = wht.wht_affine_backward(dy, x, torch.from_numpy(inp.alpha).cuda(), dx=nan_filled(N, d, "f32"))
    torch.cuda.synchronize()
    rdx, rda, rdb = oracle.backward(inp.dy, inp.x, inp.alpha, "fast")
    assert_io_close(dx, rdx, "f32", f"dx N={N}")
    assert_grad_close(da, rda, f"dalpha N={N}")
    assert_grad_close(db, rdb, f"dbeta N={N}")


@pytest.mark.parametrize("d,dtype", F32 + BF16)
def test_forward_kernels_agree_across_the_size_limit(d, dtype):
    lim = routes.persistent_from(dtype, d) - 1
    assert routes.way(dtype, d, lim) in routes.ONE_PASS and routes.way(dtype, d, lim + 37) in routes.PERSISTENT
    N = lim + 37
    print(f"[wave] forward limit d={d} {dtype} N={lim} and N={N}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(d)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.empty(N, d, device="cuda").normal_(generator=gen).to(tdt)
    a = torch.empty(d, device="cuda").uniform_(0.5, 1.5, generator=gen)
    b = torch.empty(d, device="cuda").normal_(0.0, 0.02, generator=gen)
    y_few = wht.wht_affine_forward(x[:lim], a, b, y=nan_filled(lim, d, dtype))
    y_all = wht.wht_affine_forward(x, a, b, y=nan_filled(N, d, dtype))
    torch.cuda.synchronize()
    bits = torch.int16 if dtype == "bf16" else torch.int32
    assert torch.equal(y_few.view(bits), y_all[:lim].view(bits))
    tail = x[lim - 3:].cpu()
    host = tail.view(torch.int16).numpy().view(np.uint16) if dtype == "bf16" else tail.numpy()
    ref = oracle.forward(np.ascontiguousarray(host), a.cpu().numpy(), b.cpu().numpy(), "fast")
    assert_io_close(y_all[lim - 3:], ref, dtype, f"y d={d}")
