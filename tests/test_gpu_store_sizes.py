"""The sizes at which a call changes how its results are written (plain stores, through L2, streamed), how many token
groups a workgroup of the one-pass forward kernel takes, and which forward kernel runs.  The arithmetic on a token is the
same everywhere, so a call on either side of such a size gives, row for row and bit for bit, what calls of less than
1 MiB on its rows give (plain stores, one group); no row behind the last is touched; in place as out of place."""
import pytest
import torch

import paper_2603_08343_amd as wht
import routes

pytestmark = pytest.mark.gpu

MIB = 1 << 20
CASES = [(d, "bf16") for d in (32, 64, 128, 256, 512, 1024, 2048, 4096, 8192, 16384, 768, 1536, 3072, 6144, 12288)] + \
        [(d, "f32") for d in (32, 64, 256, 1024, 2048, 4096, 8192)]
# MiB at which how dx is written, or how rows of 12 * 2^m are read, changes at some width
BACKWARD = (1, 2, 2.5, 4, 4.2, 6.3, 7.9, 8, 8.3, 9.5, 10.3, 10.4, 12, 18, 24, 32, 36, 40, 46, 56, 80, 84, 136)


def _once(d, dtype):
    """MiB of x at which this width changes its forward route, up to where y goes through L2 or not on the persistent kernel."""
    return sorted({mib for out in routes.OUTS for mib, _ in routes.steps(dtype, d, out) if 0 < mib <= 48})


def _large(d, dtype):
    """MiB at which the persistent forward kernel and the backward kernels change how they write, and what is read."""
    steps = {mib for mib, w in routes.steps(dtype, d) if w in routes.PERSISTENT}
    return sorted(steps | set(BACKWARD))


def _inputs(N, d, dtype):
    gen = torch.Generator(device="cuda").manual_seed(N + d)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x, g = (torch.empty(N, d, dtype=tdt, device="cuda").normal_(generator=gen) for _ in range(2))
    return x, g, torch.rand(d, device="cuda", generator=gen) + 0.5, torch.randn(d, device="cuda", generator=gen)


def _guarded(like, N):
    """N rows to write and one behind them, all NaN."""
    buf = torch.full((N + 1, like.shape[1]), float("nan"), dtype=like.dtype, device="cuda")
    return buf, buf[:N]


def _around(mib, row, group):
    """Row counts on both sides of the size, and a ragged last group beyond it."""
    at = int(mib * MIB) // row
    return sorted({at - 1, at, at + 1, at + group + 1})


def _pieces(N, row):
    step = max(1, (MIB - 1) // row)
    return [slice(lo, min(N, lo + step)) for lo in range(0, N, step)]


@pytest.mark.parametrize("d,dtype", CASES)
def test_forward_rows_on_both_sides_of_every_size(d, dtype):
    row = d * (2 if dtype == "bf16" else 4)
    sizes = _once(d, dtype)
    top = max(_around(sizes[-1], row, 16))
    x, r, a, b = _inputs(top, d, dtype)
    ref, ref_r, ref_s = torch.empty_like(x), torch.empty_like(x), torch.empty(top, device="cuda")
    for part in _pieces(top, row):
        ref[part] = wht.wht_affine_forward(x[part], a, b)
        ref_r[part], ref_s[part] = wht.wht_affine_forward_residual_stats(x[part], a, b, r[part])
    for mib in sizes:
        for N in _around(mib, row, 16):
            print(f"[sizes] d={d} {dtype} N={N} ({N * row / MIB:.2f} MiB)", flush=True)
            for resid, stats, want in ((None, False, ref), (r, False, ref_r), (r, True, ref_r)):
                buf, y = _guarded(x, N)
                if stats:
                    _, s = wht.wht_affine_forward_residual_stats(x[:N], a, b, resid[:N], y=y)
                    # the same squares in another order: up to log2(d) + 7 float32 roundings
                    assert bool(((s - ref_s[:N]).abs() <= 21 * 2.0 ** -24 * ref_s[:N]).all())
                elif resid is not None:
                    wht.wht_affine_forward_residual(x[:N], a, b, resid[:N], y=y)
                else:
                    wht.wht_affine_forward(x[:N], a, b, y=y)
                assert torch.equal(y, want[:N]) and bool(torch.isnan(buf[N]).all())
        same, onto = x[:N].clone(), r[:N].clone()
        wht.wht_affine_forward(same, a, b, y=same)
        wht.wht_affine_forward_residual(x[:N], a, b, onto, y=onto)
        assert torch.equal(same, ref[:N]) and torch.equal(onto, ref_r[:N])


@pytest.mark.parametrize("d,dtype", CASES)
def test_large_rows_on_both_sides_of_every_size(d, dtype):
    row = d * (2 if dtype == "bf16" else 4)
    sizes = _large(d, dtype)
    top = max(_around(sizes[-1], row, 16))
    x, g, a, b = _inputs(top, d, dtype)
    ref, ref_dx = torch.empty_like(x), torch.empty_like(x)
    for part in _pieces(top, row):
        ref[part] = wht.wht_affine_forward(x[part], a, b)
        ref_dx[part] = wht.wht_affine_backward(g[part], None, a, want_param_grads=False)[0]
    for mib in sizes:
        for N in _around(mib, row, 16)[1::2]:
            print(f"[sizes] d={d} {dtype} N={N} ({N * row / MIB:.2f} MiB)", flush=True)
            buf, out = _guarded(x, N)
            wht.wht_affine_forward(x[:N], a, b, y=out)
            assert torch.equal(out, ref[:N]) and bool(torch.isnan(buf[N]).all())
            buf, out = _guarded(x, N)
            wht.wht_affine_backward(g[:N], None, a, dx=out, want_param_grads=False)
            assert torch.equal(out, ref_dx[:N]) and bool(torch.isnan(buf[N]).all())
            buf, out = _guarded(x, N)
            da, db = wht.wht_affine_backward(g[:N], x[:N], a, dx=out)[1:]
            assert torch.equal(out, ref_dx[:N]) and bool(torch.isnan(buf[N]).all())
            again = wht.wht_affine_backward(g[:N], x[:N], a, want_dx=False)[1:]
            assert torch.equal(da, again[0]) and torch.equal(db, again[1])
        onto = g[:N].clone()
        wht.wht_affine_backward(onto, x[:N], a, dx=onto)
        assert torch.equal(onto, ref_dx[:N])


@pytest.mark.parametrize("d", [768, 1536, 3072, 6144, 12288])
def test_large_residual_rows_of_twelve(d):
    """The residual calls of rows of 12 * 2^m where x stops being kept in the cache and where y stops going through L2."""
    row = 2 * d
    top = max(_around(136, row, 16))
    x, r, a, b = _inputs(top, d, "bf16")
    ref = torch.empty_like(x)
    for part in _pieces(top, row):
        ref[part] = wht.wht_affine_forward_residual(x[part], a, b, r[part])
    for mib in (48, 56, 136):
        for N in _around(mib, row, 16):
            print(f"[sizes] residual d={d} N={N} ({N * row / MIB:.2f} MiB)", flush=True)
            for call in (wht.wht_affine_forward_residual, wht.wht_affine_forward_residual_stats):
                buf, y = _guarded(x, N)
                call(x[:N], a, b, r[:N], y=y)
                assert torch.equal(y, ref[:N]) and bool(torch.isnan(buf[N]).all())
        onto = r[:N].clone()
        wht.wht_affine_forward_residual(x[:N], a, b, onto, y=onto)
        assert torch.equal(onto, ref[:N])
