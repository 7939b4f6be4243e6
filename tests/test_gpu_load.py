"""Loading: embeddings whose rows are padded on the device go up in pieces of 64 MB; every row arrives, at the pieces' edges too."""
import numpy as np
import pytest


from harness import gpu_step, load_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [100, 129])
def test_rows_at_the_edges_of_the_pieces(H):
    at_once = (64 << 20) // (4 * H)
    V = 2 * at_once + 3
    rng = np.random.default_rng(H)
    edges = np.array([0, 1, at_once - 1, at_once, at_once + 1, 2 * at_once - 1, 2 * at_once, V - 1])
    prev = np.concatenate([edges, rng.integers(0, V, 40)]).astype(np.int32)
    U = np.full((V, H), 7.0, np.float32)                       # a row that went astray saturates every unit
    U[prev] = rng.normal(0, 0.3, (len(prev), H))
    small = 50                                                 # few output words: only the embeddings are many
    model = {"U": U, "W": rng.normal(0, 0.05, (H, H)).astype(np.float32),
             "O": np.zeros((H, V), np.float32), "bias": np.full(V, -1e4, np.float32)}
    model["O"][:, :small], model["bias"][:small] = rng.normal(0, 0.1, (H, small)), 0.0
    m = load_model(model, "f32", len(prev))
    h_in = rng.uniform(0, 1, (len(prev), H)).astype(np.float32)
    query = rng.integers(0, small, (len(prev), 2)).astype(np.int32)
    h, lp = gpu_step(m, prev, h_in, query)
    a = U[prev].astype(np.float64) + h_in.astype(np.float64) @ model["W"].astype(np.float64).T
    ref = 1.0 / (1.0 + np.exp(-a))
    assert np.max(np.abs(h - ref)) <= 2e-6                     # a quarter of some tens of roundings of sums below 2
    z = ref @ model["O"][:, :small].astype(np.float64)
    want = np.take_along_axis(z, query.astype(np.int64), 1) - np.log(np.exp(z).sum(1))[:, None]
    assert np.max(np.abs(lp - want)) <= 1e-5
    assert m.last_error() == 0
    m.close()
