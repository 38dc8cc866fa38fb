"""The density refresh of bf16 keys with many new rows (dot products on the matrix cores, near pairs by differences): edges of its
16-row and 16-key tiles, 32-key turns and 2048-key workgroups, pairs all far, some near and nearly all near (where it turns to
differences throughout), duplicates, and both sides of the line to the other form.  Against the oracle's density of the grown cloud."""
import numpy as np
import pytest

from paper_2601_01298_amd import synthetic as syn
from _util import to_device

pytestmark = pytest.mark.gpu

# An exponent d^2 / (2 sigma^2) below 40 (what is beyond adds nothing to a sum of at least 1) from a d^2 that is off by at most
# 2^-21 of itself (a far pair: 2^-23 of the norms, which are at most four times d^2), and the roundings of the sums: 4e-5 of a
# kernel value at that end, 2e-6 where values count (exponents below 4).
TOL = 5e-6


def cloud(kind, H, L, m, d, seed):
    rng = np.random.default_rng(seed)
    K = 2.0 * rng.standard_normal((H, 8, d))[:, rng.integers(0, 8, L)] + 0.5 * rng.standard_normal((H, L, d))
    if kind == "far":
        K[:, L - m:] = 2.0 * rng.standard_normal((H, m, d))
    elif kind == "offset":
        K += 30.0
    elif kind == "copies":
        K[:, L - m:] = K[:, :1]
    return syn.round_to_bf16(K.astype(np.float32))


@pytest.mark.parametrize("d,m", [(64, 7), (64, 8), (64, 15), (64, 16), (64, 17), (64, 32), (128, 3), (128, 4), (128, 5), (128, 16), (128, 31)])
@pytest.mark.parametrize("kind", ["far", "near", "offset", "copies"])
@pytest.mark.parametrize("L", [37, 50, 64, 2047, 2049, 2100])
def test_refresh_with_many_new_rows(d, m, kind, L):
    from oracle import ws_oracle as oracle
    from paper_2601_01298_amd import binding as ws
    H = 2
    K = cloud(kind, H, L, m, d, L + 7 * m + d)
    sigma = [float(syn.bandwidth(K[h])) for h in range(H)]
    old = np.stack([oracle.density(K[h, :L - m], sigma[h]) for h in range(H)]).astype(np.float32)
    got = ws.ws_synapse_density_append(to_device(K, "bf16"), m, sigma, to_device(old, "f32")).cpu().numpy()
    for h in range(H):
        assert np.abs(got[h] / oracle.density(K[h], sigma[h]) - 1).max() <= TOL


@pytest.mark.parametrize("d,m", [(64, 1), (64, 3), (64, 32), (128, 1), (128, 7), (128, 32)])
@pytest.mark.parametrize("L", [37, 63, 64, 2049, 2100])
def test_refresh_of_fp32_keys(d, m, L):
    """The sums of a lane group dealt out to its lanes: groups of 16 and 32 lanes, turns and tiles that end anywhere."""
    from oracle import ws_oracle as oracle
    from paper_2601_01298_amd import binding as ws
    K = cloud("near", 2, L, m, d, L + 7 * m + d)
    sigma = [float(syn.bandwidth(K[h])) for h in range(2)]
    old = np.stack([oracle.density(K[h, :L - m], sigma[h]) for h in range(2)]).astype(np.float32)
    got = ws.ws_synapse_density_append(to_device(K, "f32"), m, sigma, to_device(old, "f32")).cpu().numpy()
    for h in range(2):
        assert np.abs(got[h] / oracle.density(K[h], sigma[h]) - 1).max() <= TOL


def test_a_bandwidth_that_underflows_the_scale():
    """Every kernel value is 1, also where rows are missing from the last tile of 16."""
    import torch
    from paper_2601_01298_amd import binding as ws
    K = torch.randn((1, 100, 64), device="cuda").to(torch.bfloat16)
    got = ws.ws_synapse_density_append(K, 9, [1.0e19], torch.ones((1, 91), device="cuda"))
    assert torch.equal(got, torch.ones_like(got))
