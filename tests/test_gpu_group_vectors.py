"""Grouping and lookup by one workgroup where a thread's share changes (1, 2 or 4 ids), ends inside a vector or is not
16-byte aligned, and ids that want the same slots; against numbering by first appearance on the host."""
import numpy as np
import pytest
import torch

import paper_2007_11794_amd as rn

from harness import DEV

pytestmark = pytest.mark.gpu


def first_appearance(keys):
    _, first, inv = np.unique(keys, return_index=True, return_inverse=True)
    order = np.argsort(first)
    rank = np.empty(len(order), np.int64)
    rank[order] = np.arange(len(order))
    return first[order], rank[inv]


def id_hash(k):
    """As in device_utils.h."""
    m = np.uint64(0xFFFFFFFF)
    x = (k >> np.uint64(32)) * np.uint64(0x9E3779B1) & m
    x = (k + (x ^ (x >> np.uint64(16)))) & m
    x ^= x >> np.uint64(16)
    x = x * np.uint64(0x7FEB352D) & m
    return x ^ (x >> np.uint64(15))


@pytest.mark.parametrize("N", [1, 3, 1023, 1025, 2047, 2048, 2049, 2051, 3073, 4093, 4096])
def test_groups_at_the_ends_of_vectors(N):
    rng = np.random.default_rng(N)
    pool = rng.integers(0, 2 ** 64, max(1, N // 3), dtype=np.uint64)
    pool[0] = np.uint64(0xFFFFFFFFFFFFFFFF)
    keys = pool[rng.integers(0, len(pool), N)]
    rep_o, inv_o = first_appearance(keys)
    for shift in (0, 1, 3):
        ids = torch.zeros(N + 4, dtype=torch.int64, device=DEV)[shift:shift + N]
        ids.copy_(torch.from_numpy(keys.view(np.int64)))
        rep, inv = (torch.full((N + 8,), -5, dtype=torch.int32, device=DEV) for _ in range(2))
        nu = torch.zeros(1, dtype=torch.int32, device=DEV)
        ws = torch.empty(rn.rnnlm_dedup_workspace_bytes(N), dtype=torch.uint8, device=DEV)
        rn.rnnlm_dedup(ids, rep[shift:shift + N], inv[shift:shift + N], nu, ws)
        assert int(nu.item()) == len(rep_o)
        assert np.array_equal(rep.cpu().numpy()[shift:shift + len(rep_o)], rep_o)
        got = inv.cpu().numpy()
        assert np.array_equal(got[shift:shift + N], inv_o)
        assert np.all(got[:shift] == -5) and np.all(got[shift + N:] == -5)


def test_ids_that_want_the_same_slot():
    rng = np.random.default_rng(11)
    keys = rng.integers(0, 2 ** 64, 4 << 20, dtype=np.uint64)
    same = keys[(id_hash(keys) & np.uint64(8191)) == 77][:400]         # of the largest of these tables, so of the smaller ones too
    assert len(same) == 400
    for n in (400, 1500, 5000):                                        # one id a thread, two, the form beyond 4096
        ids = same[rng.integers(0, 400, n)]
        rep_o, inv_o = first_appearance(ids)
        rep, inv = (torch.full((n,), -5, dtype=torch.int32, device=DEV) for _ in range(2))
        nu = torch.zeros(1, dtype=torch.int32, device=DEV)
        ws = torch.empty(rn.rnnlm_dedup_workspace_bytes(n), dtype=torch.uint8, device=DEV)
        rn.rnnlm_dedup(torch.from_numpy(ids.view(np.int64)).to(DEV), rep, inv, nu, ws)
        assert int(nu.item()) == len(rep_o)
        assert np.array_equal(rep.cpu().numpy()[:len(rep_o)], rep_o) and np.array_equal(inv.cpu().numpy(), inv_o)


@pytest.mark.parametrize("capacity", [100000, 6000, 1500])
def test_indices_in_order_of_first_appearance(capacity):
    """Every share of a thread, rounds of the lookup one after the other, stores that fill up in the middle of one."""
    rng = np.random.default_rng(capacity)
    pool = rng.uniform(0, 1, (20000, 4)).astype(np.float32)
    t = rn.rnnlm_index_create(4, capacity, 7168)
    known, fresh = {}, 0
    for N, new in ((1, 1), (1025, 700), (2050, 1023), (2600, 1025), (4096, 2049), (7168, 4500), (4096, 0), (1024, 1024)):
        sel = np.concatenate([np.arange(fresh, fresh + new), rng.integers(0, fresh + new, N - new)])
        fresh += new
        sel = sel[rng.permutation(N)]
        want = np.full(N, 0xFFFFFFFF, np.uint32)
        for i, s in enumerate(sel):
            if s not in known and len(known) < capacity:
                known[s] = len(known)
            want[i] = known.get(s, 0xFFFFFFFF)
        index = torch.zeros(N, dtype=torch.int32, device=DEV)
        rn.rnnlm_index_intern(t, torch.zeros(N, dtype=torch.int32, device=DEV), torch.from_numpy(pool[sel]).to(DEV), index)
        assert np.array_equal(index.cpu().numpy().view(np.uint32), want), (capacity, N, new)
    assert t.stats()["entries"] == len(known)
    t.close()
