"""Rows of 12 * 2^m elements at the sizes where their schedule can go wrong: token counts that leave a wave of 768
(two tokens) half or wholly empty, both sides of the few-token limit and of the sizes at which the cache policy
changes, and one token of such a pair with an infinity or a NaN, which the matrix-core products multiply by zeros
on the way.  Elementwise against the oracle with the bounds of parity.py; the two sides of a limit bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_08343_amd as wht
import routes
from paper_2603_08343_amd import synth
from parity import assert_grad_close, assert_io_close, nan_filled, to_gpu

pytestmark = pytest.mark.gpu

@pytest.mark.parametrize("d,N", [(768, n) for n in (1, 2, 3, 4, 5, 8, 9, 23, 24, 25, 47, 4099)] +
                         [(1536, 5), (1536, 2053), (3072, 3), (3072, 1025), (6144, 2), (6144, 517), (12288, 2), (12288, 259)])
def test_every_output_at_partial_waves(d, N):
    print(f"[twelve] d={d} N={N}", flush=True)
    inp = synth.make_inputs(N, d, "bf16", seed=d + N)
    x, dy = to_gpu(inp.x, "bf16"), to_gpu(inp.dy, "bf16")
    a, b = torch.from_numpy(inp.alpha).cuda(), torch.from_numpy(inp.beta).cuda()
    y = wht.wht_affine_forward(x, a, b, y=nan_filled(N, d, "bf16"))
    yr, ss = wht.wht_affine_forward_residual_stats(x, a, b, dy)
    dx, da, db = wht.wht_affine_backward(dy, x, a, dx=nan_filled(N, d, "bf16"))
    only_dx = wht.wht_affine_backward(dy, None, a, want_param_grads=False)[0]
    only_da, only_db = wht.wht_affine_backward(dy, x, a, want_dx=False)[1:]
    torch.cuda.synchronize()
    assert_io_close(y, oracle.forward(inp.x, inp.alpha, inp.beta, "fast"), "bf16", "y")
    ref, ref_ss = oracle.forward_residual_stats(inp.x, inp.alpha, inp.beta, inp.dy, "fast")
    assert_io_close(yr, ref, "bf16", "y with residual")
    assert np.max(np.abs(ss.double().cpu().numpy() - ref_ss) / ref_ss) <= 1e-5
    rdx, rda, rdb = oracle.backward(inp.dy, inp.x, inp.alpha, "fast")
    assert_io_close(dx, rdx, "bf16", "dx")
    assert_grad_close(da, rda, "dalpha")
    assert_grad_close(db, rdb, "dbeta")
    assert torch.equal(dx, only_dx) and torch.equal(da, only_da) and torch.equal(db, only_db)


@pytest.mark.parametrize("d", [768, 1536, 3072, 6144, 12288])
def test_rows_are_the_same_on_both_sides_of_every_limit(d):
    # where the persistent forward kernel takes over, and the MiB of a tensor at which a cache policy changes: backward 32, dx alone
    # 46 and 84, forward 80 (with the residual 48 or 56), all 136
    few = {routes.persistent_from("bf16", d, out) - 1 for out in routes.OUTS}
    for N, back in [(n, False) for n in sorted(few)] + [((mib << 20) // (2 * d), mib == 32) for mib in (32, 46, 48, 56, 80, 84, 136)]:
        print(f"[twelve] d={d} N={N}", flush=True)
        gen = torch.Generator(device="cuda").manual_seed(N)
        x = torch.empty(N + 1, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
        dy = torch.empty_like(x).normal_(generator=gen)
        a, b = torch.rand(d, device="cuda", generator=gen) + 0.5, torch.randn(d, device="cuda", generator=gen)
        calls = [lambda n: wht.wht_affine_forward(x[:n], a, b), lambda n: wht.wht_affine_forward_residual(x[:n], a, b, dy[:n]),
                 lambda n: wht.wht_affine_backward(dy[:n], None, a, want_param_grads=False)[0]]
        if back:
            calls = [lambda n: wht.wht_affine_backward(dy[:n], x[:n], a)[0]]
        for call in calls:
            low, high = call(N), call(N + 1)
            assert torch.equal(low, high[:N]) and bool(torch.isfinite(high).all())
        if back:
            # the same sums in another grouping of at most 512 partial sums: float32 rounding, 1e-6 of the largest
            g0, g1 = wht.wht_affine_backward(dy[:N], x[:N], a)[1:], wht.wht_affine_backward(dy, x, a)[1:]
            z = wht.wht_affine_forward(x[N:], torch.ones_like(a), torch.zeros_like(b)).float()[0]
            last = dy[N].float()
            # z is rounded to bfloat16 here: 2^-9 of |dy z| per column
            assert bool(((g1[0] - g0[0] - last * z).abs() <= 2.0 ** -8 * (last * z).abs() + 1e-6 * g0[0].abs().max()).all())
            assert bool(((g1[1] - g0[1] - last).abs() <= 1e-6 * g0[1].abs().max()).all())


@pytest.mark.parametrize("d,N", [(768, n) for n in (1, 2, 5, 300, 512, 513, 1023, 1024, 1025, 1365, 1366, 4097)] +
                         [(1536, n) for n in (1, 3, 200, 256, 257, 512, 513, 682, 683, 2049)] + [(3072, n) for n in (1, 200, 682, 683, 1025)])
def test_forward_in_place_is_the_forward_out_of_place(d, N):
    # no wave stores what another has still to fetch: bit for bit
    print(f"[twelve] in place d={d} N={N}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(d + N)
    x = torch.empty(N, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    resid = torch.empty_like(x).normal_(generator=gen)
    a, b = torch.rand(d, device="cuda", generator=gen) + 0.5, torch.randn(d, device="cuda", generator=gen)
    y, yr = wht.wht_affine_forward(x, a, b), wht.wht_affine_forward_residual(x, a, b, resid)
    ys, ss = wht.wht_affine_forward_residual_stats(x, a, b, resid)
    assert torch.equal(yr, ys)
    for _ in range(20):
        same = [x.clone() for _ in range(3)]
        wht.wht_affine_forward(same[0], a, b, y=same[0])
        wht.wht_affine_forward_residual(same[1], a, b, resid, y=same[1])
        _, s1 = wht.wht_affine_forward_residual_stats(same[2], a, b, resid, y=same[2])
        onto = resid.clone()
        wht.wht_affine_forward_residual(x, a, b, onto, y=onto)
        assert torch.equal(same[0], y) and torch.equal(same[1], yr) and torch.equal(same[2], ys) and torch.equal(s1, ss)
        assert torch.equal(onto, yr)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("N,row", [(2, 0), (2, 1), (9, 4), (9, 8), (4098, 2049)])
def test_a_pair_of_768_keeps_a_non_finite_row_to_itself(N, row, value):
    d = 768
    print(f"[twelve] non-finite N={N} row={row} {value}", flush=True)
    inp = synth.make_inputs(N, d, "bf16", seed=N + row)
    x, dy = to_gpu(inp.x, "bf16"), to_gpu(inp.dy, "bf16")
    a, b = torch.from_numpy(inp.alpha).cuda(), torch.from_numpy(inp.beta).cuda()
    rest = np.setdiff1d(np.arange(N), [row])
    at = torch.from_numpy(rest).cuda()
    for k in (5, 600):                                            # a block of vectors 0, 1 and one of vector 2
        xk, gk = x.clone(), dy.clone()
        xk[row, k] = value
        gk[row, k] = value
        y = wht.wht_affine_forward(xk, a, b)
        yr, ss = wht.wht_affine_forward_residual_stats(xk, a, b, dy)
        dx = wht.wht_affine_backward(gk, x, a)[0]
        torch.cuda.synchronize()
        for got, ref in ((y, oracle.forward(inp.x, inp.alpha, inp.beta, "fast")),
                         (yr, oracle.forward_residual(inp.x, inp.alpha, inp.beta, inp.dy, "fast")),
                         (dx, oracle.backward(inp.dy, inp.x, inp.alpha, "fast")[0])):
            assert not bool(torch.isfinite(got[row].float()).any())
            assert_io_close(got[at], ref[rest], "bf16", f"k={k}")
        assert not bool(torch.isfinite(ss[row])) and bool(torch.isfinite(ss[at]).all())
