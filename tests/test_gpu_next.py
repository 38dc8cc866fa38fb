"""GPU parity of the steps next to the hot path, through the C ABI, element by element against the
CPU oracle on the same seeded inputs: attention-mass density proxy, density refresh after the
context grew, validation gate, RoPE-rotated injection into the cache."""
import numpy as np
import pytest

from paper_2601_01298_amd import synthetic as syn
from _util import TIE_TOL, check_indices, to_device

pytestmark = pytest.mark.gpu

MASS_TOL = 1e-4      # relative, on A: fp32 dot products of d terms feed an exponential
RHO_TOL = {"bf16": 5e-5, "f32": 1e-5}
GATE_TOL = 1e-5      # absolute, on a cosine


@pytest.fixture(scope="module")
def ws():
    import torch
    from paper_2601_01298_amd import binding
    assert torch.cuda.is_available()
    binding.lib()
    return binding


def variant(cfg, **kw):
    return syn.small_variant(syn.WORKLOADS[cfg], **kw)


def torch_dtype(dtype):
    import torch
    return torch.bfloat16 if dtype == "bf16" else torch.float32


# ------------------------------------------------------------------ attention mass
@pytest.mark.parametrize("cfg,G,Hkv,g,L", [
    (1, 1, 1, 1, 512),          # fp32, one head
    (2, 2, 4, 1, 4096),         # bf16, two layers of 4 heads
    (2, 1, 3, 2, 5000),         # grouped queries, ragged tile tail
    (5, 2, 2, 4, 3000),         # d = 128, 4 query heads per KV head
    (4, 1, 2, 8, 700),          # 8 query heads per KV head, a single short tile
    (1, 3, 2, 3, 2049),         # fp32, group size that is not a power of two, one row past a tile
])
def test_attention_mass(ws, oracle, cfg, G, Hkv, g, L):
    import torch
    w = variant(cfg, H=G * Hkv, Hq=G * Hkv * g, L=L)
    K = np.stack([syn.cloud(w, h, syn.TENSOR_K) for h in range(w.H)])
    Q = syn.main_query(w)
    Kd, Qd = to_device(K, w.dtype), to_device(Q, w.dtype)
    A = ws.ws_synapse_attention_mass(Kd, Qd, G, as_density=False).cpu().numpy()
    R = ws.ws_synapse_attention_mass(Kd, Qd, G, as_density=True).cpu().numpy()
    Hq = Hkv * g
    worst = 0.0
    for grp in range(G):
        ref = oracle.attention_mass(K[grp * Hkv:(grp + 1) * Hkv], Q[grp * Hq:(grp + 1) * Hq])
        assert abs(ref.sum() - Hq) < 1e-9
        for hk in range(Hkv):
            got = A[grp * Hkv + hk].astype(np.float64)
            big = ref > 1e-12 * ref.max()
            worst = max(worst, np.abs(got[big] / ref[big] - 1).max())
            assert np.abs(got[~big]).max(initial=0.0) <= 1e-11 * ref.max()
            rho_ref = oracle.mass_to_density(ref)
            assert np.abs(R[grp * Hkv + hk][big] / rho_ref[big] - 1).max() <= MASS_TOL
            assert np.array_equal(A[grp * Hkv + hk], A[grp * Hkv])          # every KV head gets the group's row
    print(f"attention mass cfg{cfg} G={G} Hkv={Hkv} g={g} L={L}: max rel err {worst:.2e}")
    assert worst <= MASS_TOL


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("g", [3, 4, 5, 8])
@pytest.mark.parametrize("L", [1, 15, 17, 64, 1023, 1024, 1025, 2049])
def test_attention_mass_on_the_matrix_cores(ws, oracle, d, g, L):
    """bf16 keys with three and more query heads per KV head: both instances of the kernel, group sizes below an instance's,
    the edges of its 16-key tiles and 1024-key workgroups; two groups of two KV heads."""
    w = variant(5 if d == 128 else 2, H=4, Hq=4 * g, L=L)
    K = np.stack([syn.cloud(w, h, syn.TENSOR_K) for h in range(4)])
    Q = syn.main_query(w)
    A = ws.ws_synapse_attention_mass(to_device(K, "bf16"), to_device(Q, "bf16"), 2, as_density=False).cpu().numpy()
    for grp in range(2):
        ref = oracle.attention_mass(K[2 * grp:2 * grp + 2], Q[2 * grp * g:(2 * grp + 2) * g])
        big = ref > 1e-12 * ref.max()
        assert np.abs(A[2 * grp][big] / ref[big] - 1).max() <= MASS_TOL
        assert np.abs(A[2 * grp][~big]).max(initial=0.0) <= 1e-11 * ref.max()
        assert np.array_equal(A[2 * grp], A[2 * grp + 1])


@pytest.mark.parametrize("d,g,L", [(64, 3, 9000), (64, 8, 5000), (128, 4, 4097)])
def test_attention_mass_in_a_workspace_of_an_earlier_size(ws, oracle, d, g, L):
    """A caller may have kept the size it was told when a query head had one (max, sum) pair per 2048 tokens: accepted, and
    nothing beyond it is written; one byte less is refused."""
    import torch
    w = variant(5 if d == 128 else 2, H=2, Hq=2 * g, L=L)
    K = np.stack([syn.cloud(w, h, syn.TENSOR_K) for h in range(2)])
    Q = syn.main_query(w)
    up = lambda x: (x + 255) // 256 * 256
    n = up(4 * w.Hq * L) + up(8 * w.Hq * ((L + 2047) // 2048))
    space = torch.full((n + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    out = torch.empty((2, L), device="cuda")
    Kd, Qd = to_device(K, "bf16"), to_device(Q, "bf16")
    call = lambda size: ws.lib().ws_synapse_attention_mass(Kd.data_ptr(), Qd.data_ptr(), ws.WS_BF16, 1, 2, w.Hq, L, d, 0.0, 0,
                                                           out.data_ptr(), space.data_ptr(), size, None)
    assert call(n - 1) == ws.WS_ERR_WORKSPACE
    torch.cuda.synchronize()
    assert call(n) == ws.WS_OK
    torch.cuda.synchronize()
    assert (space[n:] == 0x5A).all()
    ref = oracle.attention_mass(K, Q)
    big = ref > 1e-12 * ref.max()
    assert np.abs(out.cpu().numpy()[:, big] / ref[big] - 1).max() <= MASS_TOL


@pytest.mark.parametrize("dtype,d,g", [("bf16", 64, 1), ("bf16", 64, 4), ("bf16", 128, 8), ("f32", 128, 2)])
def test_attention_mass_far_below_the_maximum(ws, oracle, dtype, d, g):
    """One token at a logit near 60 and 2000 near 0.  What the maximum's own rounding does is common to the others; what is
    left between them is the rounding of logits below 1 (2^-25 each), of the exponential and of the sum (2^-23 each): the
    exponents may not be rounded at the size of their distance to the maximum (2^-18)."""
    L = 2001
    rng = np.random.default_rng(d + g)
    Q = syn.round_to_bf16(rng.uniform(0.5, 1.0, (g, d)).astype(np.float32))
    K = syn.round_to_bf16((rng.standard_normal((1, L, d)) * 0.05).astype(np.float32))
    K[0, 700] = syn.round_to_bf16(np.full(d, 60.0 / (0.75 * np.sqrt(d)), dtype=np.float32))
    A = ws.ws_synapse_attention_mass(to_device(K, dtype), to_device(Q, dtype), 1, as_density=False).cpu().numpy()[0]
    ref = oracle.attention_mass(K, Q)
    rest = np.arange(L) != 700
    r = A[rest].astype(np.float64) / ref[rest]
    spread = np.abs(r / np.median(r) - 1).max()
    print(f"{dtype} d={d} g={g}: spread {spread:.2e}, common {abs(np.median(r) - 1):.1e}")
    assert spread <= 6e-7


def test_attention_mass_feeds_the_selection(ws, oracle):
    """The proxy in place of the kernel density: select on 1/A must follow the oracle's greedy rule on the
    oracle's 1/A (near-tie protocol, since A of far-away tokens underflows to equal values)."""
    w = variant(2, H=4, Hq=4, L=2048, k=41)
    K = np.stack([syn.cloud(w, h, syn.TENSOR_K) for h in range(w.H)])
    Q = syn.main_query(w)
    Kd = to_device(K, w.dtype)
    rho = ws.ws_synapse_attention_mass(Kd, to_device(Q, w.dtype), 1)
    idx = ws.ws_synapse_select(Kd, rho, w.k, w.alpha).cpu().numpy()
    rho_ref = oracle.mass_to_density(oracle.attention_mass(K, Q))
    for h in range(w.H):
        ref, _, gap = oracle.select(K[h], rho_ref, w.k, w.alpha)
        forks = check_indices(oracle, K[h], rho_ref, w.k, w.alpha, idx[h], ref)
        print(f"mass->select head {h}: steps below tie tolerance {(gap < TIE_TOL).sum()}, forks {forks}")


# ------------------------------------------------------------------ density refresh
@pytest.mark.parametrize("cfg,H,L,m", [
    (1, 1, 512, 1),
    (1, 2, 700, 5),
    (2, 3, 4096, 1),
    (2, 2, 4100, 32),           # the most rows one call takes; new rows straddle a tile boundary
    (4, 2, 3000, 7),            # d = 128
    (3, 2, 2049, 2),
])
def test_density_append(ws, oracle, cfg, H, L, m):
    w = variant(cfg, H=H, Hq=H, L=L)
    K = np.stack([syn.cloud(w, h, syn.TENSOR_K) for h in range(H)])
    sigma = [float(syn.bandwidth(K[h])) for h in range(H)]
    Kd = to_device(K, w.dtype)
    rho_old = ws.ws_synapse_density(Kd[:, :L - m].contiguous(), sigma)
    rho_new = ws.ws_synapse_density_append(Kd, m, sigma, rho_old).cpu().numpy()
    worst = 0.0
    for h in range(H):
        ref = oracle.density(K[h], sigma[h])
        worst = max(worst, np.abs(rho_new[h] / ref - 1).max())
    print(f"density append cfg{cfg} H={H} L={L} m={m}: max rel err {worst:.2e}")
    assert worst <= RHO_TOL[w.dtype]


def test_density_append_many_heads(ws, oracle):
    """More heads than one launch of the sweep takes (their scales travel as a kernel argument, 768 at a time):
    heads on both sides of the seam against the oracle, every head against the full density of the library."""
    import torch
    H, L, m = 771, 300, 2
    w = variant(2, H=H, Hq=H, L=L)
    K = np.stack([syn.cloud(w, h, syn.TENSOR_K) for h in range(H)])
    sigma = [float(syn.bandwidth(K[h])) for h in range(H)]
    Kd = to_device(K, w.dtype)
    rho_old = ws.ws_synapse_density(Kd[:, :L - m].contiguous(), sigma)
    rho_new = ws.ws_synapse_density_append(Kd, m, sigma, rho_old)
    full = ws.ws_synapse_density(Kd, sigma)
    assert float((rho_new / full - 1).abs().max()) <= 2 * RHO_TOL[w.dtype]
    rho_new = rho_new.cpu().numpy()
    worst = max(np.abs(rho_new[h] / oracle.density(K[h], sigma[h]) - 1).max() for h in (0, 1, 767, 768, 769, 770))
    print(f"density append across the launch seam (H={H}): max rel err {worst:.2e}")
    assert worst <= RHO_TOL[w.dtype]


def test_density_append_repeated_steps(ws, oracle):
    """Forty decode steps of one row each, chained, against the oracle's density of the final cloud."""
    w = variant(2, H=2, Hq=2, L=1500)
    K = np.stack([syn.cloud(w, h, syn.TENSOR_K) for h in range(w.H)])
    sigma = [float(syn.bandwidth(K[h])) for h in range(w.H)]
    Kd = to_device(K, w.dtype)
    L0 = w.L - 40
    rho = ws.ws_synapse_density(Kd[:, :L0].contiguous(), sigma)
    for L in range(L0 + 1, w.L + 1):
        rho = ws.ws_synapse_density_append(Kd[:, :L].contiguous(), 1, sigma, rho)
    rho = rho.cpu().numpy()
    worst = max(np.abs(rho[h] / oracle.density(K[h], sigma[h]) - 1).max() for h in range(w.H))
    print(f"40 chained refreshes: max rel err {worst:.2e}")
    assert worst <= RHO_TOL[w.dtype]


# ------------------------------------------------------------------ validation gate
@pytest.mark.parametrize("dtype,N,dm", [("bf16", 100, 896), ("f32", 37, 896), ("bf16", 5, 1000), ("f32", 9, 33),
                                        ("bf16", 1000, 4096), ("bf16", 3, 7)])
def test_gate(ws, oracle, dtype, N, dm):
    h, T = syn.hidden_states(N, dm, dtype)
    theta = 0.5
    score, accept = ws.ws_synapse_gate(to_device(h, dtype), to_device(T, dtype), theta)
    score, accept = score.cpu().numpy(), accept.cpu().numpy()
    ref, acc_ref = oracle.gate(h, T, theta)
    err = np.abs(score - ref).max()
    print(f"gate {dtype} N={N} dm={dm}: max abs err {err:.2e}, accepted {accept.sum()} of {N}")
    assert err <= GATE_TOL
    assert score[0] == 0.0 and accept[0] == 0                                    # the zero thought
    assert np.array_equal(accept, (score >= np.float32(theta)).astype(np.int32))   # decision on the fp32 score
    clear = np.abs(ref - theta) > GATE_TOL
    assert np.array_equal(accept[clear], acc_ref[clear])                         # and the oracle's wherever it is clear
    assert 0 < accept.sum() < N or N < 4


# ------------------------------------------------------------------ injection
@pytest.mark.parametrize("cfg,H,L,Lcap,m", [(1, 1, 512, 600, 5), (2, 3, 100, 164, 64), (4, 2, 0, 16, 16),
                                            (5, 2, 1000, 1001, 1)])
def test_inject(ws, oracle, cfg, H, L, Lcap, m):
    import torch
    w = variant(cfg, H=H, Hq=H, L=max(L, 1))
    base = 1.0e6
    Kn, Vn, pos = syn.thought_rows(w, m)
    rng = np.random.default_rng(5)
    Kc0 = rng.standard_normal((H, Lcap, w.d)).astype(np.float32)
    Vc0 = rng.standard_normal((H, Lcap, w.d)).astype(np.float32)
    if w.dtype == "bf16":
        Kc0, Vc0 = syn.round_to_bf16(Kc0), syn.round_to_bf16(Vc0)
    Kc, Vc = to_device(Kc0, w.dtype), to_device(Vc0, w.dtype)
    used = ws.ws_synapse_inject(Kc, Vc, L, to_device(Kn, w.dtype), to_device(Vn, w.dtype),
                                torch.from_numpy(pos).cuda(), base)
    assert used == L + m
    Kc, Vc = Kc.float().cpu().numpy(), Vc.float().cpu().numpy()
    keep = np.ones(Lcap, dtype=bool)
    keep[L:L + m] = False
    assert np.array_equal(Kc[:, keep], Kc0[:, keep]) and np.array_equal(Vc[:, keep], Vc0[:, keep])
    assert np.array_equal(Vc[:, L:L + m], Vn)
    worst = 0.0
    for h in range(H):
        ref = oracle.rope(Kn[h], pos, base)
        got = Kc[h, L:L + m].astype(np.float64)
        half = w.d // 2
        mag = np.hypot(Kn[h][:, :half], Kn[h][:, half:]).astype(np.float64)      # rotation keeps each pair's radius
        mag = np.concatenate([mag, mag], axis=1)
        # fp32 rotation, then (bf16) one rounding of the result: half a unit in the last place of the radius
        tol = (2.0 ** -8 if w.dtype == "bf16" else 4e-7) * mag + 1e-30
        worst = max(worst, (np.abs(got - ref) / tol).max())
    print(f"inject cfg{cfg} H={H} L={L} m={m}: worst error / tolerance {worst:.3f}")
    assert worst <= 1.0
