"""The selection at the sizes where the one-workgroup kernel takes over from the others and at the edges of its row slots,
and on clouds whose far point is picked at most steps (the prediction of the next D_max and the grouped exact evaluation of
the resident kernel): picks equal the oracle's, or differ from them only in near-ties (both within 1e-5 of the best score,
the rule of the parity tests)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def check(K, rho, k, alpha, dtype, kernel="auto", heads=None):
    import torch
    from oracle import ws_oracle as oracle
    from paper_2601_01298_amd import binding as ws
    ws.lib()
    Kd = torch.from_numpy(K).to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda()
    score = torch.empty((K.shape[0], k), dtype=torch.float32, device="cuda")
    idx = ws.ws_synapse_select(Kd, torch.from_numpy(rho).cuda(), k, alpha, kernel=kernel, score_out=score)[0].cpu().numpy()
    score = score.cpu().numpy()
    for h in range(K.shape[0] if heads is None else heads):
        assert len(set(idx[h])) == k and idx[h].min() >= 0 and idx[h].max() < K.shape[1]
        ref, ref_score, _ = oracle.select(K[h], rho[h], k, alpha)
        if not np.array_equal(idx[h], ref):
            forks, _, deficit = oracle.select_verify(K[h], rho[h], k, alpha, idx[h])
            assert forks >= 0 and deficit.max() <= 1e-5
        # the winning scores of one chain are the other's up to the tie rule, whichever of two tied keys was taken
        same = np.cumprod(idx[h] == ref).astype(bool)
        assert np.allclose(score[h][same], ref_score[same], rtol=2e-5, atol=0)
    assert np.isfinite(score).all()
    return idx, score


def data(H, L, d, dtype, seed, far=0.0):
    from paper_2601_01298_amd import synthetic as syn
    rng = np.random.default_rng(seed)
    K = (2.0 * rng.standard_normal((H, 8, d)))[:, rng.integers(0, 8, L)] + 0.5 * rng.standard_normal((H, L, d))
    rho = rng.uniform(0.05, 1.0, (H, L))
    out = rng.random((H, L)) < far
    K[out] = rng.uniform(-8, 8, (int(out.sum()), d))
    rho[out] = 0.05
    K = K.astype(np.float32)
    return syn.round_to_bf16(K) if dtype == "bf16" else K, rho.astype(np.float32)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,L", [(64, 1), (64, 2), (64, 128), (64, 129), (64, 257), (64, 512), (64, 513), (64, 1023), (64, 1024),
                                 (64, 1025), (128, 3), (128, 255), (128, 257), (128, 512), (128, 513)])
def test_small_heads(d, L, dtype):
    for alpha in (0.0, 0.5, 1.0):
        check(*data(3, L, d, dtype, 7 * L + d), min(L, 12), alpha, dtype)


def test_small_head_to_the_last_key():
    K, rho = data(2, 130, 64, "f32", 5)
    K[:, 64:] = K[:, :66]                 # duplicates: D_max reaches 0 with keys left
    check(K, rho, 130, 0.5, "f32")


def test_more_small_heads_than_compute_units():
    check(*data(300, 200, 64, "f32", 9), 4, 0.5, "f32")


# heads in the call -> key rows per lane in registers and in LDS (and more than 32 workgroups per head: a wide instance)
@pytest.mark.parametrize("d,H,L,split", [(64, 2, 1500, (1, 0)), (64, 2, 3000, (1, 0)), (64, 40, 4096, (2, 0)), (64, 96, 4096, (4, 0)),
                                         (64, 600, 1000, (4, 0)), (64, 2, 40000, (6, 2)), (128, 2, 1200, (1, 0)), (128, 2, 6000, (1, 0)),
                                         (128, 40, 4096, (2, 0)), (128, 520, 512, (2, 0)), (128, 72, 4096, (3, 1)), (128, 2, 40000, (3, 1))])
@pytest.mark.parametrize("far", [0.02, 0.3])
def test_far_points_picked_first(d, H, L, split, far):
    """Every split of the resident kernel on clouds whose far point is picked at most steps: D_max without the pick carried
    through the exchange (or, with one workgroup per head, through LDS), and strips that fill up and are refilled.  Heads are
    copies of two clouds: the two against the oracle, the copies against them."""
    from paper_2601_01298_amd import binding as ws
    plan = ws.ws_synapse_select_plan("resident", ws.WS_BF16, H, L, d)
    assert (plan.rows_in_registers, plan.rows_in_lds) == split, "this head count no longer selects the split"
    K, rho = data(2, L, d, "bf16", L, far)
    copies = np.arange(H) % 2
    idx, score = check(K[copies], rho[copies], 60, 0.5, "bf16", "resident", heads=2)
    assert np.array_equal(idx, idx[copies]) and np.array_equal(score, score[copies])
