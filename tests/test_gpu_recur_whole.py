"""Hidden update with all operands on their way at once, against the oracle: ends of rows inside a piece of four units, hidden
sizes at the limits of its kernels, row counts where 32 units a workgroup become 64, two workgroups share a compute unit and the
ring takes over, the count known on the host, to the device only, and found by the launch itself."""
import numpy as np
import pytest
import torch

import oracle
import paper_2007_11794_amd as rn

from harness import DEV, load_model
from test_gpu_recur import V, model_of

pytestmark = pytest.mark.gpu


def check(m, model, dtype, H, prev, h_in, out, rows):
    ref = oracle.step(model, prev[rows], h_in[rows], np.zeros((len(rows), 1), np.int32))["h_out"]
    # as in test_gpu_recur
    assert np.max(np.abs(out[rows] - ref)) <= (2e-6 if dtype == "f32" else 1e-5)
    assert m.last_error() == 0


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H,B", [(1, 5), (3, 40), (4, 33), (5, 31), (6, 64), (7, 65), (129, 97), (254, 1025), (256, 1024), (256, 1025), (257, 32), (320, 700), (384, 512), (384, 641),
                                 (509, 513), (511, 1), (512, 513), (512, 1025), (512, 2048), (512, 2049), (513, 260), (766, 257), (767, 300), (768, 512), (640, 256), (638, 769), (640, 768), (770, 513), (896, 250),
                                 (1021, 129), (1024, 257), (1024, 513)])
def test_rows_known_on_the_host(H, B, dtype):
    rng = np.random.default_rng(H * 5000 + B)
    model = model_of(rng, H, dtype)
    m = load_model(model, dtype, B)
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    rows = np.unique(np.concatenate([np.arange(0, B, 61), np.arange(max(0, B - 34), B)]))
    for shift in (0, 1):                                       # h_in and h_out 16-byte aligned (where rows can be), 4-byte aligned
        buf_in = torch.full((B * H + 4,), float("nan"), device=DEV)            # nothing beyond a row counts
        buf_out = torch.full((B * H + 4,), float("nan"), device=DEV)
        h_t, out = buf_in[shift:shift + B * H].view(B, H), buf_out[shift:shift + B * H].view(B, H)
        h_t.copy_(torch.from_numpy(h_in))
        rn.rnnlm_step(m, torch.from_numpy(prev).to(DEV), h_t, torch.zeros((B, 1), dtype=torch.int32, device=DEV), out, torch.zeros((B, 1), device=DEV))
        got = buf_out.cpu().numpy()
        assert np.isnan(got[:shift]).all() and np.isnan(got[shift + B * H:]).all()
        check(m, model, dtype, H, prev, h_in, got[shift:shift + B * H].reshape(B, H), rows)
    m.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H,N,unique", [(130, 200, 77), (200, 1000, 1000), (512, 1024, 513), (333, 1024, 1024), (1024, 256, 256),       # grouped by the launch
                                        (64, 1500, 33), (333, 1500, 512), (512, 2300, 512), (512, 2300, 513), (512, 2300, 1024), (512, 2300, 1025),
                                        (512, 2300, 2048), (512, 2300, 2049), (257, 1100, 1), (1024, 1100, 40)])                          # in front of it
def test_rows_found_on_the_device(H, N, unique, dtype):
    rng = np.random.default_rng(H * 7 + N + unique)
    model = model_of(rng, H, dtype)
    m = load_model(model, dtype, N)
    src = np.concatenate([np.arange(unique), rng.integers(0, unique, N - unique)])[rng.permutation(N)]
    prev, h_in = rng.integers(0, V, unique).astype(np.int32)[src], rng.uniform(0, 1, (unique, H)).astype(np.float32)[src]
    order = np.sort(np.unique(src, return_index=True)[1])                      # first appearances
    shift = N % 2                                                              # not 16-byte aligned
    h_t = torch.zeros(N * H + 4, device=DEV)[shift:shift + N * H].view(N, H)
    h_t.copy_(torch.from_numpy(h_in))
    h_out = torch.full((N, H), float("nan"), device=DEV)
    i32 = dict(dtype=torch.int32, device=DEV)
    rep, inv, nu = torch.zeros(N, **i32), torch.zeros(N, **i32), torch.zeros(1, **i32)
    ws = torch.empty(rn.rnnlm_dedup_workspace_bytes(N), dtype=torch.uint8, device=DEV)
    rn.rnnlm_step_dedup(m, torch.from_numpy(src.astype(np.int64) * 77 + 1).to(DEV), torch.from_numpy(prev).to(DEV), h_t, torch.zeros((N, 1), **i32), rep, inv, nu,
                        h_out, torch.zeros((N, 1), device=DEV), ws)
    assert int(nu.item()) == unique and np.array_equal(rep.cpu().numpy()[:unique], order)
    got = h_out.cpu().numpy()
    assert np.isnan(got[unique:]).all()
    check(m, model, dtype, H, prev[order], h_in[order], got[:unique], np.unique(np.concatenate([np.arange(0, unique, 61), np.arange(max(0, unique - 34), unique)])))
    m.close()
