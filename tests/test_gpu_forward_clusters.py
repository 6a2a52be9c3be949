"""The forward kernel's deal of token groups to clusters of workgroups, on both sides of the number of rounds from
which it is used (32, for rows of 12 * 2^m elements 48; 512 workgroups), with a last region that is short and one
that is ragged: bit for bit the rows of calls that are too short for it, which other tests hold against the oracle."""
import pytest
import torch

import paper_2603_08343_amd as wht

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,dtype,first", [(4096, torch.bfloat16, 32 * 512 * 2), (8192, torch.bfloat16, 32 * 512),
                                           (4096, torch.float32, 32 * 512), (1024, torch.float32, 32 * 512 * 4),
                                           (3072, torch.bfloat16, 48 * 512 * 2), (6144, torch.bfloat16, 48 * 512)])
def test_clusters_compute_the_rows_of_the_plain_walk(d, dtype, first):
    gen = torch.Generator(device="cuda").manual_seed(d)
    top = first + 61
    x = torch.empty(top, d, dtype=dtype, device="cuda").normal_(generator=gen)
    resid = torch.empty_like(x).normal_(generator=gen)
    a, b = torch.rand(d, device="cuda", generator=gen) + 0.5, torch.randn(d, device="cuda", generator=gen)
    step = first // 4
    plain = torch.cat([wht.wht_affine_forward(x[i:i + step], a, b) for i in range(0, top, step)])
    plain_r = torch.cat([wht.wht_affine_forward_residual(x[i:i + step], a, b, resid[i:i + step]) for i in range(0, top, step)])
    for N in (first - 1, first, first + 1, top):
        print(f"[clusters] d={d} N={N}", flush=True)
        y = torch.full_like(x, float("nan"))
        wht.wht_affine_forward(x[:N], a, b, y=y[:N])
        assert torch.equal(y[:N], plain[:N]) and bool(torch.isnan(y[N:]).all())
        y.fill_(float("nan"))
        wht.wht_affine_forward_residual(x[:N], a, b, resid[:N], y=y[:N])
        assert torch.equal(y[:N], plain_r[:N]) and bool(torch.isnan(y[N:]).all())
