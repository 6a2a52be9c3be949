"""The rules of dispatch (csrc/wht_route.h) on the host: what they say is whole for every width, dtype and output."""
import pytest

import routes

WIDTHS = [("bf16", 1 << n) for n in range(5, 15)] + [("bf16", 12 << m) for m in range(6, 11)] + [("f32", 1 << n) for n in range(5, 14)]


@pytest.mark.parametrize("dtype,d", WIDTHS)
def test_every_size_has_a_way(dtype, d):
    for out in routes.OUTS:
        for butterfly in (False, True):
            s = routes.steps(dtype, d, out, butterfly)
            mib = [m for m, _ in s]
            assert mib[0] == 0 and mib == sorted(set(mib)), (out, s)
            assert s[0][1] == "plain" and s[-1][1] == "stream", (out, s)
            assert routes.way(dtype, d, routes.persistent_from(dtype, d, out, butterfly), out, butterfly) in routes.PERSISTENT
            for i, (m, w) in enumerate(s):
                n = routes.tokens(dtype, d, m)
                assert routes.way(dtype, d, n, out, butterfly) == w or routes.tokens(dtype, d, s[min(i + 1, len(s) - 1)][0]) <= n
                if i and n > 1:
                    assert routes.way(dtype, d, n - 1, out, butterfly) != w or s[i - 1][1] == w


# What was measured at these sizes, streamed and through L2, stands beside dx_through.
@pytest.mark.parametrize("dtype,d,mib,grads,through", [
    ("f32", 8192, 30, False, False), ("f32", 8192, 60, False, True), ("f32", 2048, 36, False, False), ("bf16", 512, 11, False, False),
    ("bf16", 4096, 34, False, False), ("bf16", 1024, 36, False, True), ("bf16", 1024, 5, False, False), ("f32", 4096, 30, False, True),
    ("bf16", 16384, 100, False, False), ("bf16", 64, 6, False, False), ("bf16", 64, 9, False, True), ("bf16", 2048, 1.5, False, False), ("f32", 128, 9, False, True), ("f32", 1024, 9, False, False),
    ("bf16", 768, 40, False, True), ("bf16", 768, 75, False, False), ("bf16", 12288, 75, False, False), ("bf16", 3072, 100, False, True),
    ("f32", 256, 10, True, False), ("bf16", 64, 7, True, False), ("bf16", 32, 30, True, False), ("bf16", 128, 100, True, True),
    ("f32", 512, 12, True, False), ("f32", 512, 20, True, True), ("f32", 1024, 1.5, True, False), ("bf16", 4096, 5, True, True),
    ("bf16", 2048, 0.5, True, False), ("bf16", 2048, 0.5, False, False), ("bf16", 1024, 160, True, False), ("bf16", 6144, 20, True, True)])
def test_dx_goes_where_it_was_faster(dtype, d, mib, grads, through):
    assert routes.dx_through(dtype, d, routes.tokens(dtype, d, mib), grads) is through


@pytest.mark.parametrize("dtype,d,dx,store", [("bf16", 64, True, "plain"), ("f32", 128, False, "plain"), ("f32", 256, True, "plain"),
                                              ("f32", 256, False, "through"), ("bf16", 512, True, "through"), ("f32", 4096, False, "stream"),
                                              ("f32", 4096, True, "through"), ("bf16", 4096, False, "through"), ("bf16", 12288, True, "through")])
def test_partial_rows_are_written_as_was_faster(dtype, d, dx, store):
    assert routes.sums_store(dtype, d, dx) == store


# Both sides of what was measured at these sizes stand beside forward_route; the sizes are those at which another way was slower.
@pytest.mark.parametrize("dtype,d,out,mib,way", [
    ("f32", 2048, "y", 30, "plain"), ("f32", 2048, "y", 20, "stream"), ("f32", 2048, "stats", 30, "plain"), ("f32", 64, "stats", 12, "plain"), ("f32", 512, "stats", 12, "through"), ("f32", 8192, "stats", 70, "stream"),
    ("bf16", 1024, "y", 14, "through"), ("bf16", 1024, "y", 30, "through"), ("bf16", 1024, "stats", 12, "plain"), ("bf16", 2048, "stats", 16, "plain"),
    ("bf16", 4096, "y", 28, "stream"), ("bf16", 4096, "stats", 25, "stream"), ("bf16", 8192, "resid", 7.5, "plain"), ("bf16", 16384, "stats", 70, "stream"),
    ("bf16", 1536, "stats", 20, "stream"), ("bf16", 3072, "stats", 3.4, "through"), ("bf16", 6144, "y", 14, "stream"), ("bf16", 12288, "stats", 15, "through"),
    ("bf16", 12288, "stats", 27, "stream")])
def test_forward_takes_the_way_that_was_faster(dtype, d, out, mib, way):
    assert routes.way(dtype, d, routes.tokens(dtype, d, mib), out) == way
