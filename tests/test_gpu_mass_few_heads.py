"""The attention mass of bf16 keys with one and two query heads per KV head, on both sides of the line between its two forms
(512 tiles of 1024 keys), at the edges of the matrix-core form's 16-key tiles and 1024-key workgroups."""
import numpy as np
import pytest

from paper_2601_01298_amd import synthetic as syn
from _util import to_device

pytestmark = pytest.mark.gpu

MASS_TOL = 1e-4         # relative on A: the tolerance of the other attention-mass tests


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("g", [1, 2])
@pytest.mark.parametrize("H,L", [(2, 1), (2, 15), (2, 17), (3, 1023), (2, 1024), (2, 1025), (1, 5001), (255, 2048), (256, 2049)])
def test_one_and_two_query_heads(d, g, H, L):
    from oracle import ws_oracle as oracle
    from paper_2601_01298_amd import binding as ws
    rng = np.random.default_rng(H * L + d + g)
    K = syn.round_to_bf16(rng.standard_normal((H, L, d)).astype(np.float32))
    Q = syn.round_to_bf16(rng.standard_normal((H * g, d)).astype(np.float32))
    A = ws.ws_synapse_attention_mass(to_device(K, "bf16"), to_device(Q, "bf16"), H, as_density=False).cpu().numpy()
    for h in sorted({0, H // 2, H - 1}):
        ref = oracle.attention_mass(K[h:h + 1], Q[h * g:(h + 1) * g])
        big = ref > 1e-12 * ref.max()
        assert np.abs(A[h][big] / ref[big] - 1).max() <= MASS_TOL
        assert np.abs(A[h][~big]).max(initial=0.0) <= 1e-11 * ref.max()
