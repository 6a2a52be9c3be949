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
            first = next(i for i, (_, w) in enumerate(s) if w in routes.PERSISTENT)      # from there on only persistent
            assert all(w in routes.PERSISTENT for _, w in s[first:]), (out, s)
            for i, (m, w) in enumerate(s):
                n = routes.tokens(dtype, d, m)
                assert routes.way(dtype, d, n, out, butterfly) == w or routes.tokens(dtype, d, s[min(i + 1, len(s) - 1)][0]) <= n
                if i and n > 1:
                    assert routes.way(dtype, d, n - 1, out, butterfly) != w or s[i - 1][1] == w
