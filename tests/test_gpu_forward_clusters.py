"""The forward kernel's deal of token groups to clusters of workgroups, on both sides of the number of rounds from
which it is used (20, for rows of 12 * 2^m elements 48; 512 workgroups), with a last region that is short and one
that is ragged: bit for bit the rows of calls that are too short for it, which other tests hold against the oracle."""
import pytest
import torch

import paper_2603_08343_amd as wht

pytestmark = pytest.mark.gpu


# width, dtype, rounds from which token groups are dealt, tokens of a group
@pytest.mark.parametrize("d,dtype,rounds,G", [(4096, torch.bfloat16, 20, 2), (8192, torch.bfloat16, 20, 1), (4096, torch.float32, 20, 1),
                                              (1024, torch.float32, 20, 4), (3072, torch.bfloat16, 48, 2), (6144, torch.bfloat16, 48, 1)])
def test_clusters_compute_the_rows_of_the_plain_walk(d, dtype, rounds, G):
    first = (rounds * 512 - 1) * G + 1                    # the first count of that many rounds, its last group ragged where G > 1
    gen = torch.Generator(device="cuda").manual_seed(d)
    top = first + 61 + G
    x = torch.empty(top, d, dtype=dtype, device="cuda").normal_(generator=gen)
    resid = torch.empty_like(x).normal_(generator=gen)
    a, b = torch.rand(d, device="cuda", generator=gen) + 0.5, torch.randn(d, device="cuda", generator=gen)
    step = first // 4
    plain = torch.cat([wht.wht_affine_forward(x[i:i + step], a, b) for i in range(0, top, step)])
    plain_r = torch.cat([wht.wht_affine_forward_residual(x[i:i + step], a, b, resid[i:i + step]) for i in range(0, top, step)])
    for N in (first - 1, first, first + G - 1, first + G, top):
        print(f"[clusters] d={d} N={N}", flush=True)
        y = torch.full_like(x, float("nan"))
        wht.wht_affine_forward(x[:N], a, b, y=y[:N])
        assert torch.equal(y[:N], plain[:N]) and bool(torch.isnan(y[N:]).all())
        y.fill_(float("nan"))
        wht.wht_affine_forward_residual(x[:N], a, b, resid[:N], y=y[:N])
        assert torch.equal(y[:N], plain_r[:N]) and bool(torch.isnan(y[N:]).all())
