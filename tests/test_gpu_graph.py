"""A whole gradient step (forward with storage, residual, reverse sweep) captured in a HIP
graph and replayed: every replay, with eager work and synchronisations in between, must
reproduce the eager result bitwise (the library records no memset nodes: it clears memory
with its own fill kernel)."""
import numpy as np
import pytest
import torch

import paper_2304_05592_amd as A
import workloads as W
from helpers import gpu_inputs, make_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", [A.Storage(A.STORE_FULL), A.Storage(A.STORE_CHECKPOINT, 3),
                                     A.Storage(A.STORE_FULL, 0, A.PREC_BF16)])
def test_graph_replays_match_eager(storage):
    wl = W.small_2d(nshot=2)
    plan = make_plan(wl, storage=storage)
    m, q = gpu_inputs(wl, plan, background=True)
    m_true, _ = gpu_inputs(wl, plan)
    ws = plan.workspace()
    d_obs = plan.forward(m_true, q, ws=ws)
    d = torch.empty_like(d_obs)
    r = torch.empty_like(d_obs)
    g = torch.empty(plan.layout.m_size, dtype=torch.float64, device="cuda")

    def step():
        plan.forward(m, q, d=d, keep=True, ws=ws)
        _, loss = A.residual(d, d_obs, r=r)
        plan.backward(m, q, r, g=g, v=None, ws=ws)
        return loss

    loss = step()
    torch.cuda.synchronize()
    g_ref, loss_ref = g.clone(), loss.clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        loss_g = step()
    torch.cuda.synchronize()
    for it in range(3):
        g.zero_()
        d.zero_()
        _ = plan.forward(m_true, q, ws=plan.workspace())   # unrelated eager work between replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(g, g_ref), it
        assert torch.equal(loss_g, loss_ref), it


@pytest.mark.parametrize("shots", [2, 60])
def test_graph_replays_after_a_change_of_the_fusion_mode(shots):
    """A graph holds the addresses of the plan's tables: a change of the fusion mode after the capture, with eager
    calls in the other modes in between, leaves every replay bitwise right (narrow tiles, and enough shots for
    128-column ones)."""
    wl = W.small_2d(nshot=2) if shots == 2 else W.small_2d(nz=40, windows=[230] * shots, T_per_shot=[60.0] * shots, nrec=9)
    plan = make_plan(wl, storage=A.Storage(A.STORE_FULL))
    m, q = gpu_inputs(wl, plan)
    dd = torch.randn(plan.layout.d_size, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    dm = 0.001 * m
    ws = plan.workspace()
    g = torch.empty(plan.layout.m_size, dtype=torch.float64, device="cuda")
    d, jd = torch.empty_like(dd), torch.empty_like(dd)

    def calls():
        plan.forward(m, q, d=d, keep=True, ws=ws)
        plan.backward(m, q, dd, g=g, ws=ws)
        plan.born(m, q, dm, dd=jd, ws=ws)

    calls()
    torch.cuda.synchronize()
    ref = [t.clone() for t in (g, d, jd)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls()
    for mode in (A.FUSE_NONE, A.FUSE_FORWARD, A.FUSE_ADJOINT, A.FUSE_BOTH):
        plan.set_fusion(mode)
        for run in (calls, graph.replay):
            for t in (g, d, jd):
                t.zero_()
            run()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip((g, d, jd), ref)), (mode, run)
