"""Which steps are a single launch: what rnnlm_one_launch says against the nodes of the captured step, on both sides of the rules."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2007_11794_amd as rn

from harness import DEV, load_model
from test_gpu_hs_step import make as make_tree
from test_gpu_step_few import inputs, make

pytestmark = pytest.mark.gpu


def launches(step):
    """Nodes of the graph that one call records."""
    step()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        step()
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


class Step:
    def __init__(self, m, V, H, B, N, K):
        prev, h_in, query, row = inputs(V, H, B, N, K)
        self.m, self.N = m, N
        self.prev, self.h_in, self.query, self.row = (torch.from_numpy(x).to(DEV) for x in (prev, h_in, query, row))
        self.h_out, self.lp, self.base = torch.zeros((B, H), device=DEV), torch.zeros((N, K), device=DEV), torch.zeros((N, K), device=DEV)
        self.ids = torch.arange(N, device=DEV) // 2
        self.rep, self.inv, self.nu = (torch.zeros(n, dtype=torch.int32, device=DEV) for n in (N, N, 1))
        self.ws = torch.empty(rn.rnnlm_dedup_workspace_bytes(N), dtype=torch.uint8, device=DEV)

    def rows(self, mapped=False, tree=False):
        call = rn.rnnlm_hs_step if tree else rn.rnnlm_step
        call(self.m, self.prev, self.h_in, self.query, self.h_out, self.lp, row_of_query=self.row if mapped else None)

    def grouped(self, base=None, score=None):
        rn.rnnlm_step_cached(self.m, None, self.ids, self.prev, self.h_in, self.query, self.rep, self.inv, self.nu, self.h_out,
                             self.lp if score is None else score, self.ws, base_score=base)


@pytest.mark.parametrize("dtype,V,H,B,K,one", [("f32", 1000, 64, 8, 4, True), ("f32", 1000, 64, 33, 4, False), ("f32", 1000, 129, 4, 4, False),
                                               ("bf16", 1000, 129, 4, 4, True), ("bf16", 1000, 256, 16, 4, True), ("bf16", 1000, 256, 17, 4, False),
                                               ("bf16", 1000, 257, 2, 4, False), ("bf16", 1000, 64, 2, 0, False)])
def test_rows_and_grouped(dtype, V, H, B, K, one):
    m = load_model(make(V, H, dtype), dtype, 64)
    s = Step(m, V, H, B, B, K)
    assert m.one_launch(B, B, K) == m.one_launch(0, B, K, grouped=True) == one
    assert (launches(s.rows) == 1) == one
    assert (launches(s.grouped) == 1) == one
    if one:
        assert m.one_launch(B, B, K, mapped=True) and launches(lambda: s.rows(mapped=True)) == 1
        assert launches(lambda: s.grouped(base=s.base)) == 1
        assert launches(lambda: s.grouped(base=s.lp)) > 1                   # the answers in the place of the base scores
        m.set_option(rn.OPT_OUTPROJ_KERNEL, 5)
        assert not m.one_launch(B, B, K) and launches(s.rows) > 1
    m.close()


@pytest.mark.parametrize("dtype,V,H,B,N,K,one", [("f32", 1000, 64, 8, 1, 8192, True), ("f32", 1000, 64, 8, 1, 8193, False), ("f32", 1000, 64, 8, 128, 32, True),
                                                 ("f32", 1000, 64, 8, 64, 128, True), ("f32", 1000, 64, 8, 256, 24, False), ("f32", 4000, 128, 8, 200, 40, False),
                                                 ("bf16", 8000, 256, 6, 256, 8, True), ("bf16", 8000, 256, 6, 100, 30, False), ("bf16", 8000, 256, 6, 32, 128, True),
                                                 ("bf16", 8000, 256, 6, 64, 128, False), ("bf16", 90000, 128, 4, 64, 64, True), ("bf16", 90000, 128, 4, 400, 20, False)])
def test_many_words(dtype, V, H, B, N, K, one):
    """Where the last workgroup would take longer over the words than the separate launches."""
    m = load_model(make(V, H, dtype), dtype, 512)
    s = Step(m, V, H, B, N, K)
    assert m.one_launch(B, N, K, mapped=True) == one
    assert (launches(lambda: s.rows(mapped=True)) == 1) == one
    m.close()


@pytest.mark.parametrize("dtype,V,H,B,rows,grouped", [("f32", 4000, 128, 24, True, True), ("f32", 4000, 128, 25, False, True), ("bf16", 4000, 128, 32, True, True),
                                                      ("bf16", 5000, 192, 16, True, True), ("bf16", 5000, 192, 17, False, False), ("f32", 30000, 64, 16, True, True),
                                                      ("f32", 30000, 64, 17, False, True), ("f32", 34000, 64, 8, True, True), ("f32", 34000, 64, 9, False, True),
                                                      ("f32", 42000, 128, 8, True, True), ("f32", 46000, 128, 1, False, True), ("f32", 67000, 128, 8, True, True)])
def test_rows_times_units_and_bytes(dtype, V, H, B, rows, grouped):
    """The lines of step_few_chosen, where the caller has told the rows apart and where the ids are grouped."""
    m = load_model(make(V, H, dtype), dtype, 64)
    s = Step(m, V, H, B, B, 4)
    assert m.one_launch(B, B, 4) == rows and m.one_launch(0, B, 4, grouped=True) == grouped
    assert (launches(s.rows) == 1) == rows and (launches(s.grouped) == 1) == grouped
    m.close()


@pytest.mark.parametrize("dtype,H,B,N,K,mapped,one", [("f32", 128, 512, 512, 4, False, True), ("f32", 128, 513, 513, 4, False, False), ("bf16", 128, 9, 9, 3, False, False),
                                                      ("bf16", 256, 256, 256, 6, False, True), ("bf16", 257, 9, 9, 8, False, False), ("f32", 180, 128, 256, 6, True, True),
                                                      ("f32", 180, 129, 256, 6, True, False)])
def test_tree(dtype, H, B, N, K, mapped, one):
    _, m = make_tree(H, dtype, 1024)
    s = Step(m, 1500, H, B, N, K)
    assert m.one_launch(B, N, K, mapped=mapped) == one and not m.one_launch(B, N, K, grouped=True)
    assert (launches(lambda: s.rows(mapped, tree=True)) == 1) == one
    m.close()


def test_bad_arguments():
    L = rn.lib()
    assert L.rnnlm_one_launch(None, 1, 1, 1, 0) == -1
    m = load_model(make(100, 64, "f32"), "f32", 4)
    assert [L.rnnlm_one_launch(m.handle, 1, 1, 1, form) for form in (-1, 3)] == [-1, -1]
    m.close()
