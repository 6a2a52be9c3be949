"""Infinities and NaN: they stay in the rows and columns that the definition takes them to.

A ragged last token group has slots without a token.  Nothing that such a slot reads may reach dalpha:
a product with a dy of zero keeps it out for finite values only.  In place (dx = x or dx = dy) the last
row is also being overwritten by the wave that owns it, so a slot that still read it would see either
content.  Token counts: one group and a bit, and several groups per workgroup, each leaving whole waves
and (where a wave holds several tokens) parts of a wave without a token."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_08343_amd as wht
import routes
from paper_2603_08343_amd import synth
from parity import assert_grad_close, assert_io_close, nan_filled, to_gpu

pytestmark = pytest.mark.gpu

# width, dtype, tokens of a workgroup pass, tokens of a wave
WAVE = [(64, "f32", 32, 8), (256, "f32", 16, 4), (1024, "f32", 4, 1), (2048, "f32", 4, 1), (32, "bf16", 64, 16),
        (256, "bf16", 16, 4), (512, "bf16", 8, 2)]
WIDE = [(4096, "f32", 1, 1), (8192, "f32", 1, 1)]                     # two and four waves per token
MATRIX = [(768, "bf16", 8, 2), (1024, "bf16", 4, 1), (1536, "bf16", 4, 1), (2048, "bf16", 4, 1), (4096, "bf16", 2, 1),
          (3072, "bf16", 2, 1)]


def _counts(G, W, d):
    workgroups = 1024 if d <= 64 else 512
    few = (19, 33, 91, 509) if d == 768 else ()       # few elements; from 86 on workgroups of four tokens with partial rows
    return (G + W + 1, 2 * workgroups * G + W + 1, *few)


def _params(inp):
    return torch.from_numpy(inp.alpha).cuda(), torch.from_numpy(inp.beta).cuda()


def _sylvester_signs(d, k):
    return np.array([-1.0 if bin(j & k).count("1") & 1 else 1.0 for j in range(d)])


@pytest.mark.parametrize("alias", ["x", "dy"])
@pytest.mark.parametrize("d,dtype,G,W", WAVE + MATRIX)
def test_infinite_gradient_in_the_last_row_in_place(d, dtype, G, W, alias):
    for N in _counts(G, W, d):
        print(f"[nonfinite] dx={alias} d={d} {dtype} N={N}", flush=True)
        inp = synth.make_inputs(N, d, dtype, seed=5 * d + N)
        col = d // 3
        x, dy = to_gpu(inp.x, dtype), to_gpu(inp.dy, dtype)
        a, _ = _params(inp)
        dy[N - 1, col] = float("inf")
        _, da0, db0 = wht.wht_affine_backward(dy, x, a)               # out of place
        dx, da, db = wht.wht_affine_backward(dy, x, a, dx=x if alias == "x" else dy)
        torch.cuda.synchronize()
        # the reference with a finite value there: every other column and row is the same
        inp.dy[N - 1, col] = 0
        rdx, rda, rdb = oracle.backward(inp.dy, inp.x, inp.alpha, "fast")
        rest = np.arange(d) != col
        for got, ref, name in ((da, rda, "dalpha"), (db, rdb, "dbeta")):
            assert not bool(torch.isfinite(got[col])), name
            assert_grad_close(got[torch.from_numpy(rest).cuda()], ref[rest], f"{name} d={d} N={N}")
        assert torch.equal(da.nan_to_num(7.0), da0.nan_to_num(7.0)) and torch.equal(db.nan_to_num(7.0), db0.nan_to_num(7.0))
        assert_io_close(dx[:N - 1], rdx[:N - 1], dtype, f"dx d={d} N={N}")
        assert not bool(torch.isfinite(dx[N - 1].float()).any())


@pytest.mark.parametrize("d,dtype,G,W", WAVE + WIDE)
def test_infinite_input_in_the_last_row(d, dtype, G, W):
    # z[N-1] is +-Inf in every column, so dalpha is +-Inf with the sign of dy z: NaN would be a missing
    # token's 0 * Inf
    for N in _counts(G, W, d):
        print(f"[nonfinite] x d={d} {dtype} N={N}", flush=True)
        inp = synth.make_inputs(N, d, dtype, seed=6 * d + N)
        k = d // 2 + 5
        x, dy = to_gpu(inp.x, dtype), to_gpu(inp.dy, dtype)
        a, _ = _params(inp)
        x[N - 1, k] = float("inf")
        dy[N - 1] = torch.where(dy[N - 1] == 0, torch.ones_like(dy[N - 1]), dy[N - 1])
        dx, da, db = wht.wht_affine_backward(dy, x, a, dx=nan_filled(N, d, dtype))
        torch.cuda.synchronize()
        want = np.sign(dy[N - 1].double().cpu().numpy()) * _sylvester_signs(d, k) * np.inf
        assert np.array_equal(da.cpu().numpy(), want.astype(np.float32))
        if dtype == "f32":
            inp.dy[N - 1] = dy[N - 1].cpu().numpy()
        else:
            inp.dy[N - 1] = dy[N - 1].view(torch.int16).cpu().numpy().view(np.uint16)
        rdx, _, rdb = oracle.backward(inp.dy, synth.make_inputs(N, d, dtype, seed=6 * d + N).x, inp.alpha, "fast")
        assert_io_close(dx, rdx, dtype, f"dx d={d} N={N}")
        assert_grad_close(db, rdb, f"dbeta d={d} N={N}")


@pytest.mark.parametrize("d,dtype,N", [(256, "f32", 19), (2048, "f32", 7), (8192, "f32", 5), (64, "bf16", 67), (512, "bf16", 11),
                                       (1024, "f32", 8195), (4096, "f32", 1029), (512, "bf16", 32775),
                                       (1024, "f32", "persistent"), (4096, "f32", "persistent"), (512, "bf16", "persistent")])
def test_forward_rows_with_infinity_and_nan(d, dtype, N):
    if N == "persistent":
        N = max(routes.persistent_from(dtype, d, out) for out in ("y", "stats")) + 3
        assert all(routes.way(dtype, d, N, out) in routes.PERSISTENT for out in ("y", "stats"))
    print(f"[nonfinite] forward d={d} {dtype} N={N}", flush=True)
    inp = synth.make_inputs(N, d, dtype, seed=7 * d + N)              # dy doubles as the residual stream
    x, resid = to_gpu(inp.x, dtype), to_gpu(inp.dy, dtype)
    a, b = _params(inp)
    k, inf_row, nan_row = d // 4 + 3, N - 1, N // 2
    x[inf_row, k] = float("-inf")
    x[nan_row, k] = float("nan")
    y = wht.wht_affine_forward(x, a, b)
    yr, ss = wht.wht_affine_forward_residual_stats(x, a, b, resid)
    torch.cuda.synchronize()
    ref = oracle.forward(inp.x, inp.alpha, inp.beta, "fast")
    ref_r, ref_ss = oracle.forward_residual_stats(inp.x, inp.alpha, inp.beta, inp.dy, "fast")
    rest = np.setdiff1d(np.arange(N), [inf_row, nan_row])
    at = torch.from_numpy(rest).cuda()
    want = -np.inf * _sylvester_signs(d, k)                           # alpha > 0
    for got, r in ((y, ref), (yr, ref_r)):
        assert np.array_equal(got[inf_row].double().cpu().numpy(), want)
        assert bool(torch.isnan(got[nan_row].float()).all())
        assert_io_close(got[at], r[rest], dtype, f"d={d} N={N}")
    assert float(ss[inf_row]) == float("inf") and bool(torch.isnan(ss[nan_row]))
    assert np.max(np.abs(ss[at].double().cpu().numpy() - ref_ss[rest]) / ref_ss[rest]) <= 1e-5


@pytest.mark.parametrize("d", [768, 1024, 4096])
def test_matrix_core_forward_keeps_an_infinity_in_its_row(d):
    N = 9
    print(f"[nonfinite] matrix-core forward d={d} N={N}", flush=True)
    inp = synth.make_inputs(N, d, "bf16", seed=d)
    x = to_gpu(inp.x, "bf16")
    a, b = _params(inp)
    x[4, 77] = float("inf")
    y = wht.wht_affine_forward(x, a, b)
    torch.cuda.synchronize()
    rest = np.setdiff1d(np.arange(N), [4])
    assert not bool(torch.isfinite(y[4].float()).any())
    assert_io_close(y[torch.from_numpy(rest).cuda()], oracle.forward(inp.x, inp.alpha, inp.beta, "fast")[rest], "bf16", f"d={d}")
