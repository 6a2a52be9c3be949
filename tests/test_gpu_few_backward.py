"""The backward pass of a few tokens in one launch (backward_few_kernel): a slice of 64 columns per workgroup for dalpha and
dbeta, a wave for every 16th token, up to four tokens of a wave at a time.  Every output against the oracle at token
counts around those steps and on both sides of the size up to which the kernel runs; dx bit for bit what the other
kernels give (alone, and in the place of dy or x, where the call takes them)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2603_08343_amd as wht
import routes
from paper_2603_08343_amd import synth
from parity import assert_grad_close, assert_io_close, nan_filled, to_gpu

pytestmark = pytest.mark.gpu

LIMITS = {(t, d): routes.few_elements(t, d) for t, widths in (("bf16", [1 << n for n in range(5, 15)] + [12 << m for m in range(6, 11)]),
                                                              ("f32", [1 << n for n in range(5, 14)])) for d in widths
          if routes.few_elements(t, d)}


@pytest.mark.parametrize("dtype,d", list(LIMITS))
def test_every_output_around_the_steps_and_the_limit(dtype, d):
    top = LIMITS[dtype, d] // d
    for N in sorted({1, 2, 3, 16, 17, 31, 33, 64, 65, top - 1, top, top + 1} & set(range(1, top + 2))):
        print(f"[few] d={d} {dtype} N={N}", flush=True)
        inp = synth.make_inputs(N, d, dtype, seed=d + N)
        x, dy = to_gpu(inp.x, dtype), to_gpu(inp.dy, dtype)
        a = torch.from_numpy(inp.alpha).cuda()
        buf = nan_filled(N + 1, d, dtype)
        dx, da, db = wht.wht_affine_backward(dy, x, a, dx=buf[:N])
        again = wht.wht_affine_backward(dy, x, a)
        only_dx = wht.wht_affine_backward(dy, None, a, want_param_grads=False)[0]
        only = wht.wht_affine_backward(dy, x, a, want_dx=False)[1:]
        onto_dy, onto_x = dy.clone(), x.clone()
        in_place = wht.wht_affine_backward(onto_dy, x, a, dx=onto_dy), wht.wht_affine_backward(dy, onto_x, a, dx=onto_x)
        torch.cuda.synchronize()
        rdx, rda, rdb = oracle.backward(inp.dy, inp.x, inp.alpha, "fast")
        assert_io_close(dx, rdx, dtype, "dx")
        for ga, gb in ((da, db), in_place[0][1:], in_place[1][1:]):
            assert_grad_close(ga, rda, "dalpha")
            assert_grad_close(gb, rdb, "dbeta")
        assert bool(torch.isnan(buf[N].float()).all())
        assert all(torch.equal(p, q) for p, q in zip((dx, da, db), again))
        assert torch.equal(only[0], da) and torch.equal(only[1], db)
        assert all(torch.equal(dx, t) for t in (only_dx, onto_dy, onto_x))


@pytest.mark.parametrize("dtype,d", [("bf16", 512), ("bf16", 768), ("bf16", 4096), ("bf16", 6144), ("f32", 256), ("f32", 8192)])
def test_one_hot_rows_reach_every_column(dtype, d):
    """x one-hot at column k: z = +-1/sqrt(d), so dalpha is that row of H times dy; one token at a time and all at once."""
    N = min(LIMITS[dtype, d] // d, 48)
    print(f"[few] one-hot d={d} {dtype} N={N}", flush=True)
    rng = np.random.RandomState(d)
    at = np.concatenate(([0, 1, 63, 64, d - 1], rng.randint(0, d, N)))[:N]
    x = torch.zeros(N, d, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    x[torch.arange(N), torch.from_numpy(at).cuda()] = 1.0
    dy = torch.ones_like(x)
    a, zero = torch.ones(d, device="cuda"), torch.zeros(d, device="cuda")
    rows = wht.wht_affine_forward(x.float() if dtype == "f32" else x, a, zero).double()          # +-1/sqrt(d), rounded
    da, db = wht.wht_affine_backward(dy, x, a)[1:]
    signs = torch.sign(rows).sum(0)                                                              # exact
    assert torch.equal(torch.round(da.double() * d ** 0.5), signs) and torch.equal(db, torch.full_like(db, float(N)))


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("dtype,d", [("bf16", 512), ("bf16", 768), ("bf16", 8192), ("f32", 1024)])
def test_non_finite_values_stay_where_they_belong(dtype, d, value):
    N = 11
    print(f"[few] non-finite d={d} {dtype} {value}", flush=True)
    inp = synth.make_inputs(N, d, dtype, seed=d)
    x, dy = to_gpu(inp.x, dtype), to_gpu(inp.dy, dtype)
    a = torch.from_numpy(inp.alpha).cuda()
    _, rda, rdb = oracle.backward(inp.dy, inp.x, inp.alpha, "fast")
    bad_x = x.clone()
    bad_x[10, 3] = value                                       # every z of the row, so every dalpha; no dbeta
    dx, da, db = wht.wht_affine_backward(dy, bad_x, a)
    assert not bool(torch.isfinite(da).any()) and bool(torch.isfinite(dx.float()).all())
    assert_grad_close(db, rdb, "dbeta")
    bad_dy = dy.clone()
    bad_dy[10, 3] = value                                      # one column of the sums, one row of dx
    dx, da, db = wht.wht_affine_backward(bad_dy, x, a)
    keep = torch.arange(d, device="cuda") != 3
    assert not bool(torch.isfinite(da[3])) and not bool(torch.isfinite(db[3]))
    assert bool(torch.isfinite(da[keep]).all()) and bool(torch.isfinite(db[keep]).all())
    assert not bool(torch.isfinite(dx[10].float()).any()) and bool(torch.isfinite(dx[:10].float()).all())


@pytest.mark.parametrize("dtype,d", [("bf16", 768), ("bf16", 512), ("bf16", 4096), ("f32", 1024)])
def test_sums_in_the_place_of_alpha(dtype, d):
    """dalpha or dbeta over alpha itself: another kernel's call, in a workspace of the size asked for and not a byte more."""
    code = wht.DTYPE_BF16 if dtype == "bf16" else wht.DTYPE_F32
    for N in (1, 4, 5, 8, 9, 16, 17, 32):
        inp = synth.make_inputs(N, d, dtype, seed=3 * d + N)
        x, dy = to_gpu(inp.x, dtype), to_gpu(inp.dy, dtype)
        rdx, rda, rdb = oracle.backward(inp.dy, inp.x, inp.alpha, "fast")
        need = max(16, wht.wht_affine_backward_workspace_bytes(N, d, code))
        for over in ("dalpha", "dbeta"):
            print(f"[few] over alpha d={d} {dtype} N={N} {over}", flush=True)
            a = torch.from_numpy(inp.alpha).cuda()
            room = torch.full((need + (1 << 16),), 77, dtype=torch.uint8, device="cuda")
            dx, da, db = wht.wht_affine_backward(dy, x, a, workspace=room[:need], **{over: a})
            assert (da if over == "dalpha" else db).data_ptr() == a.data_ptr()
            assert bool((room[need:] == 77).all())
            assert_io_close(dx, rdx, dtype, "dx")
            assert_grad_close(da, rda, "dalpha")
            assert_grad_close(db, rdb, "dbeta")


def _butterflies(z):
    """H_raw z in z's own precision, stage by stage."""
    n, d = z.shape
    h = 1
    while h < d:
        v = z.view(n, d // (2 * h), 2, h)
        z = torch.stack((v[:, :, 0] + v[:, :, 1], v[:, :, 0] - v[:, :, 1]), dim=2).view(n, d)
        h *= 2
    return z


@pytest.mark.parametrize("d", [1024, 2048, 4096, 8192])
def test_float32_sums_are_as_exact_as_the_butterflies(d):
    """dalpha of single float32 tokens against 64 bits: no further off than the transform done stage by stage in float32, whose
    every value is added in log2 d levels.  32 such errors are averaged (each the 2-norm over d columns, so the average varies
    by less than 1 %), and 5 % are left for the order of the lane sums; one chain over the loads is 15 % off at 4096, 31 % at 8192."""
    rng = torch.Generator().manual_seed(d)
    x, dy = torch.randn(32, d, generator=rng), torch.randn(32, d, generator=rng)
    exact = _butterflies(x.double()) * dy.double() / d ** 0.5
    plain = (_butterflies(x) * dy) * torch.tensor(1.0 / d ** 0.5)
    ones = torch.ones(d, device="cuda")
    got = torch.stack([wht.wht_affine_backward(dy[n:n + 1].cuda(), x[n:n + 1].cuda(), ones)[1].cpu() for n in range(32)])
    off = lambda t: float(((t.double() - exact).norm(dim=1) / exact.norm(dim=1)).mean())
    print(f"[few] d={d} off by {off(got):.3e}, butterflies {off(plain):.3e}", flush=True)
    assert off(got) <= 1.05 * off(plain)


def _launches(call):
    """Kernels that a call launches, counted in a captured graph."""
    hip = ctypes.CDLL("libamdhip64.so")
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    count = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


# tokens of a workgroup of the other kernels, and how many such groups one workgroup takes
@pytest.mark.parametrize("dtype,d,group,groups", [("bf16", 512, 8, 3), ("bf16", 1024, 4, 3), ("bf16", 2048, 4, 2), ("bf16", 4096, 2, 2),
                                                  ("bf16", 8192, 1, 2), ("bf16", 768, 8, 2), ("bf16", 1536, 4, 2), ("bf16", 12288, 1, 1),
                                                  ("f32", 256, 16, 3), ("f32", 512, 8, 3), ("f32", 1024, 4, 3), ("f32", 8192, 1, 1)])
def test_few_groups_over_alpha_are_one_launch(dtype, d, group, groups):
    """dalpha or dbeta over alpha: up to as many token groups as one workgroup takes in a single launch, as on buffers of its own."""
    code = wht.DTYPE_BF16 if dtype == "bf16" else wht.DTYPE_F32
    for N in (1, group, group * groups):
        print(f"[few] over alpha, one launch, d={d} {dtype} N={N}", flush=True)
        inp = synth.make_inputs(N, d, dtype, seed=5 * d + N)
        x, dy = to_gpu(inp.x, dtype), to_gpu(inp.dy, dtype)
        rdx, rda, rdb = oracle.backward(inp.dy, inp.x, inp.alpha, "fast")
        ws = torch.empty(max(16, wht.wht_affine_backward_workspace_bytes(N, d, code)), dtype=torch.uint8, device="cuda")
        for over in ("dalpha", "dbeta", None):
            a = torch.from_numpy(inp.alpha).cuda()
            out = {"dx": torch.empty_like(x), "dalpha": torch.empty_like(a), "dbeta": torch.empty_like(a), **({over: a} if over else {})}
            assert _launches(lambda: wht.wht_affine_backward(dy, x, a, workspace=ws, **out)) == 1, over     # captured, not run
            wht.wht_affine_backward(dy, x, a, workspace=ws, **out)
            assert_io_close(out["dx"], rdx, dtype, f"dx, {over} over alpha")
            assert_grad_close(out["dalpha"], rda, f"dalpha, {over} over alpha")
            assert_grad_close(out["dbeta"], rdb, f"dbeta, {over} over alpha")


@pytest.mark.parametrize("dtype,d", list(LIMITS))
def test_in_place_or_not_is_the_same_bits(dtype, d):
    """dx over dy or x: dx, dalpha and dbeta bit for bit those of a call on buffers of its own, up to behind the limit of the kernel."""
    top = LIMITS[dtype, d] // d
    for N in sorted({1, 2, 3, 4, 5, 8, 9, 12, 13, 16, 17, 24, 25, 48, top, top + 1} & set(range(1, top + 2))):
        print(f"[few] in place d={d} {dtype} N={N}", flush=True)
        inp = synth.make_inputs(N, d, dtype, seed=7 * d + N)
        x, dy, a = to_gpu(inp.x, dtype), to_gpu(inp.dy, dtype), torch.from_numpy(inp.alpha).cuda()
        apart = wht.wht_affine_backward(dy, x, a)
        onto_dy, onto_x = dy.clone(), x.clone()
        assert all(torch.equal(p, q) for p, q in zip(apart, wht.wht_affine_backward(onto_dy, x, a, dx=onto_dy)))
        assert all(torch.equal(p, q) for p, q in zip(apart, wht.wht_affine_backward(dy, onto_x, a, dx=onto_x)))
