"""The density at the sizes where its two sweeps change hands or run short: edges of the 32-row tiles, of the 128- and
256-key blocks, odd and even block counts (with an even count the block half way round is visited from both sides; the sweep
in blocks of 256 pads to an even count, so odd ones are those of the sweep in blocks of 128), counts at which several
workgroups share a row block's visits; a NaN key, which reaches every density of its head; and kernel sums
that rounding has driven to infinity, which have to come out as that."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# the density tolerances of the parity tests: 2^-23 |k|^2 / sigma^2 per kernel term, about 2e-6 at this bandwidth
TOL = {"bf16": 5e-5, "f32": 1e-5}


@pytest.fixture(scope="module")
def ws():
    from paper_2601_01298_amd import binding
    binding.lib()
    return binding


def cloud(H, L, d, dtype, seed):
    from paper_2601_01298_amd import synthetic as syn
    rng = np.random.default_rng(seed)
    centres = 2.0 * rng.standard_normal((H, 8, d))
    pick = rng.integers(0, 8, (H, L))
    K = (np.take_along_axis(centres, pick[:, :, None], axis=1) + 0.5 * rng.standard_normal((H, L, d))).astype(np.float32)
    return syn.round_to_bf16(K) if dtype == "bf16" else K


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [1, 2, 33, 128, 129, 256, 384, 511, 768, 769, 1024, 1281, 2305])
def test_density_block_edges(ws, L, d, dtype):
    import torch
    from oracle import ws_oracle as oracle
    H = 2
    K = cloud(H, L, d, dtype, 1000 * d + L)
    sigma = [float(np.float32(np.sqrt(max(K[h].var(axis=0).sum(), 1.0) / 16))) for h in range(H)]
    Kd = torch.from_numpy(K).to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda()
    rho = ws.ws_synapse_density(Kd, sigma).cpu().numpy()
    for h in range(H):
        ref = oracle.density(K[h], sigma[h])
        assert np.abs(rho[h] / ref - 1).max() <= TOL[dtype]


@pytest.mark.parametrize("L,dtype", [(200, "f32"), (2100, "f32"), (500, "bf16"), (769, "bf16"), (2100, "bf16")])
def test_nan_key_reaches_its_head(ws, L, dtype):
    import torch
    K = torch.from_numpy(cloud(2, L, 64, dtype, L)).to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda()
    K[1, L // 3, 5] = float("nan")
    rho = ws.ws_synapse_density(K, [3.0, 3.0])
    assert torch.isfinite(rho[0]).all() and torch.isnan(rho[1]).all()


@pytest.mark.parametrize("L,dtype", [(300, "f32"), (2100, "f32"), (300, "bf16"), (768, "bf16"), (769, "bf16"), (2100, "bf16")])
def test_overflowing_sums_are_infinite_and_flagged(ws, L, dtype):
    """Norms of 6e9 around a common point, differences of order 1: the exponents are rounding errors of up to several times the
    fp32 spacing there (512), of either sign, which the bandwidth of 0.01 turns into 0 or infinity.  A density is then infinite
    or a plain sum of values (never below its self term, never a number out of range, never NaN); the head beside it is not
    touched."""
    import torch
    K = cloud(2, L, 64, dtype, L)
    rng = np.random.default_rng(L)
    K[1] = 1e4 * rng.standard_normal(64) + rng.standard_normal((L, 64))
    K[1, 0] = 0.01                      # (a key near zero: the head cannot be moved to the origin exactly)
    Kd = torch.from_numpy(K).to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda()
    space = torch.empty(ws.ws_synapse_workspace_bytes(ws.WS_OP_DENSITY, ws.WS_BF16 if dtype == "bf16" else ws.WS_F32, 2, L, 64),
                        dtype=torch.uint8, device="cuda")
    rho = ws.ws_synapse_density(Kd, [3.0, 0.01], workspace=space)
    flagged, est = ws.ws_synapse_density_check(space, 2)
    assert flagged and est[1] > 2e-5 >= est[0]
    rho = rho.cpu().numpy()
    assert np.isinf(rho[1]).sum() > L // 3
    rest = rho[1, ~np.isinf(rho[1])]
    assert (rest >= 0.999 / L).all() and (rest <= 32).all()
    assert (rho[0] > 0).all() and (rho[0] <= 1).all()


@pytest.mark.parametrize("d,bound", [(64, 2.3e-7), (128, 2.5e-7)])
def test_fp32_error_on_clustered_clouds(ws, d, bound):
    """Products of fp32 keys are summed from bf16 pieces; their mean error may not grow past what fp32 products gave on these
    inputs (2.6e-7, 3.4e-7), and does not reach what it was with the norms added last (2.4e-7, 2.6e-7): 2.2e-7, 2.4e-7."""
    import torch
    from oracle import ws_oracle as oracle
    v = []
    for L in (200, 512, 700, 1500):
        K = cloud(8, L, d, "f32", d + L)
        sigma = [float(np.float32(np.sqrt(K[h].var(axis=0).sum() / 16))) for h in range(8)]
        rho = ws.ws_synapse_density(torch.from_numpy(K).cuda(), sigma).cpu().numpy()
        ref = np.stack([oracle.density(K[h], sigma[h]) for h in range(8)])
        v += [np.linalg.norm(rho[h] - ref[h]) / np.linalg.norm(ref[h]) for h in range(8)]
    print(f"d={d}: mean 2-norm error {np.mean(v):.4e}")
    assert np.mean(v) <= bound
