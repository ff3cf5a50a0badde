"""GPU test of the greedy pick: the first maximum of the logits, whatever lane, packet or round it lies in."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2311_02103_amd.runtime import DeviceModel  # noqa: E402


@pytest.mark.parametrize("V", [8, 31, 4096, 32000, 32768, 32776, 70000])
def test_greedy_pick_is_the_first_maximum(V):
    """Ties across lanes, packets and rounds; both zeros; minus infinities; NaNs, which are never the maximum (a row of NaNs only: index 0); through a
    model without layers whose head copies its input."""
    H = 64
    rng = np.random.default_rng(V)
    emb = np.zeros((V, H), np.float16)
    emb[:, 0] = 1.0                                        # after the norm every row is sqrt(H) in column 0, zero elsewhere
    for case in range(7):
        head = np.zeros((V, H), np.float16)
        head[:, 0] = rng.integers(-3, 3, V) if case == 0 else -1.0 if case == 1 else 0.0 if case == 2 else rng.standard_normal(V)
        if case == 1:
            head[V // 2:, 0] = -np.inf
        if case == 2:
            head[::2, 0] = -0.0
        if case in (4, 5):                                 # NaNs of either sign in front of, between and behind the numbers
            head[:, 0] = rng.integers(-3, 3, V) if case == 4 else -np.inf
            head[rng.permutation(V)[:max(2, V // 3)], 0] = np.nan
            head[[0, V - 1], 0] = np.nan, -np.nan
        if case == 6:
            head[:, 0] = np.nan
        m = DeviceModel([], emb.view(np.uint16), np.ones(H, np.float16).view(np.uint16), head.view(np.uint16), hidden=H, n_heads=1, n_kv_heads=1, head_dim=64,
                        ffn=64, kv_capacity=8, kv_slots=2, n_max=2, rms_eps=1e-5, rope_base=10000.0, group=32)
        logits, ids = m.step(torch.zeros(2, dtype=torch.int32, device="cuda"), [1, 1], [1, 1])
        got = logits.float().cpu().numpy()
        assert bool(np.isnan(got).any()) == (case >= 4)
        assert ids.cpu().tolist() == [0 if np.isnan(r).all() else int(np.flatnonzero(r == np.nanmax(r))[0]) for r in got], (V, case)
