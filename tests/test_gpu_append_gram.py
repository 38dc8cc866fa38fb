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
    elif kind == "split":       # the first 16 new rows far from every key, the rest near to all: each turn fills its list several times
        K += 30.0
        K[:, L - m:L - m + 16] -= 60.0
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


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("m", [17, 25, 32])
@pytest.mark.parametrize("L", [50, 2047, 2100, 6000])
def test_second_tile_of_new_rows_near(d, m, L):
    test_refresh_with_many_new_rows(d, m, "split", L)


def test_second_tile_of_new_rows_near_is_no_slower_than_direct():
    """The same at a size that fills the chip, against as many rows all near to every key, which are evaluated directly: 1.2 of its time;
    2.5 when only the first 16 rows decided whether a wave goes on that way."""
    import torch
    from paper_2601_01298_amd import binding as ws
    H, L, m, d = 96, 32768, 32, 64
    near = 20.0 + torch.randn((H, L, d), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    times = []
    for first in (0.0, 40.0):
        K = near.clone()
        K[:, L - m:L - m + 16] -= first
        K, rho = K.to(torch.bfloat16), torch.full((H, L - m), 0.5, device="cuda")
        best = float("inf")
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            ws.ws_synapse_density_append(K, m, [3.0] * H, rho)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        times.append(best)
    print(times)
    assert times[1] < 1.5 * times[0]


@pytest.mark.parametrize("m", [2, 8, 20])
def test_rows_that_are_no_numbers(m):
    """A new row with an infinity has no density, whichever form the refresh takes (its distance to itself is no number); the keys around
    it have theirs, as it is infinitely far."""
    import torch
    from paper_2601_01298_amd import binding as ws
    K = cloud("near", 1, 200, m, 64, 5)
    K[0, 200 - m, 7] = np.inf
    got = ws.ws_synapse_density_append(to_device(K, "bf16"), m, [3.0], torch.full((1, 200 - m), 0.5, device="cuda")).cpu().numpy()[0]
    assert np.isnan(got[200 - m]) and np.isfinite(np.delete(got, 200 - m)).all()
