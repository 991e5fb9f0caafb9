"""Continuous-batching server on the GPU: every request's result is the same
alone and in a mix, admission respects the HBM budget, cancellation frees a
running slot."""
import math

import numpy as np
import pytest

from oracle import oracle as O
from paper_2410_19075_amd import inputs

pytestmark = pytest.mark.gpu
FHN_PRM = [0.05, 0.5, 0.1, math.pi / 2 - 0.1]
HH_PRM = [1.0, 120.0, 36.0, 0.3, 50.0, -77.0, -54.387, 0.0, 0.0, 2.0]


@pytest.fixture(scope="module")
def nd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_19075_amd import nd as _nd
    return _nd


def cases(nd):
    rp, col, w = inputs.random_out_graph(9, 600, 12)
    sw = inputs.small_world_links(5, 1500, 10, 30)
    return [
        (nd.problem(nd.ND_KURAMOTO, nd.ND_RING, 1024, [0.0, 1.0, 1.46], radius=256),
         inputs.kuramoto_phases(1, 1024), 0.01, 150, 1),
        (nd.problem(nd.ND_FHN, nd.ND_RING, 3000, FHN_PRM, radius=1000), inputs.fhn_circle(2, 3000), 0.01, 97, 5),
        (nd.problem(nd.ND_KURAMOTO, nd.ND_RING, 5000, [0.1, 1.0, 1.3], precision=nd.ND_FP32_BULK, radius=900),
         inputs.kuramoto_phases(3, 5000), 0.01, 130, 2),
        (nd.problem(nd.ND_FHN, nd.ND_RING, 700, FHN_PRM, radius=40), inputs.fhn_circle(4, 700), 0.01, 60, 0),
        (nd.problem(nd.ND_KURAMOTO, nd.ND_CUBE3D, 12 ** 3, [0.0, 1.0, 0.8], radius=2, dims=(12, 12, 12)),
         inputs.kuramoto_phases(5, 12 ** 3), 0.05, 50, 10),
        (nd.problem(nd.ND_HH, nd.ND_CSR, 600, HH_PRM, row_ptr=rp, col=col, weight=w,
                    per_elem=inputs.hh_iapp(9, 600)), inputs.hh_state(9, 600), 0.01, 80, 0),
        (nd.problem(nd.ND_FHN, nd.ND_RING, 20000, FHN_PRM, precision=nd.ND_FP32_BULK, radius=7000),
         inputs.fhn_circle(7, 20000), 0.01, 45, 3),
        # the paper's 3D inertia model on a ball, its 2D disk, and a compressed coupling matrix
        (nd.problem(nd.ND_KURAMOTO_INERTIA, nd.ND_BALL3D, 12 ** 3, [0.0, 0.5, 0.45, 1.0, 0.05], radius=2,
                    dims=(12, 12, 12)),
         np.concatenate([inputs.kuramoto_phases(11, 12 ** 3), np.zeros(12 ** 3)]), 0.05, 40, 4),
        (nd.problem(nd.ND_KURAMOTO_INERTIA, nd.ND_BALL3D, 13 ** 3, [0.0, 0.5, 0.45, 1.0, 0.05], radius=4,
                    dims=(13, 13, 13)),  # plane-scatter form
         np.concatenate([inputs.kuramoto_phases(14, 13 ** 3), np.zeros(13 ** 3)]), 0.05, 21, 3),
        (nd.problem(nd.ND_KURAMOTO, nd.ND_DISK2D, 20 * 18, [0.0, 1.0, 0.8], radius=3, dims=(20, 18, 1)),
         inputs.kuramoto_phases(12, 20 * 18), 0.05, 33, 0),
        (nd.problem(nd.ND_FHN, nd.ND_LINKS, 1500, FHN_PRM, row_ptr=sw[0], col=sw[1]), inputs.fhn_circle(13, 1500),
         0.01, 55, 5),
    ]


def drain(nd, s, stream=None, guard=10000):
    for _ in range(guard):
        if nd.nd_server_pump(s, stream) == 0:
            return
    raise AssertionError("server did not drain")


def test_alone_equals_mix_bitwise(nd):
    cs = cases(nd)
    alone = [nd.simulate(p, y0, dt, steps, record_every=r) for p, y0, dt, steps, r in cs]
    s = nd.nd_server_create(8 << 30, max_slots=16, chunk_steps=16)
    try:
        ids = []
        for k, (p, y0, dt, steps, r) in enumerate(cs):
            ids.append(nd.nd_server_submit(s, p, y0, dt, steps, nd.observe(r, -1)))
            if k == 2:
                nd.nd_server_pump(s)  # later requests join while others run
        drain(nd, s)
        for rid, (p, y0, dt, steps, r), (ya, Ra, _) in zip(ids, cs, alone):
            info = nd.nd_server_info(s, rid)
            assert info.state == nd.ND_REQ_DONE and info.steps_done == steps
            assert info.arrival <= info.admitted <= info.finished
            y = np.empty_like(y0)
            R = np.empty(steps // r + 1) if r else None
            nd.nd_server_result(s, rid, y, R)
            assert np.array_equal(y, ya)
            if r:
                assert np.array_equal(R, Ra)
        st = nd.nd_server_stats(s)
        assert st.completed == len(cs) and st.running == 0 and st.bytes_in_use == 0
    finally:
        nd.nd_server_destroy(s)


def test_mixed_results_match_oracle(nd):
    """Small requests of the mix against the FP64 oracle (FP64 ones to 1e-12)."""
    cs = [c for c in cases(nd)[:5] if c[0].precision == 0]
    s = nd.nd_server_create(8 << 30, max_slots=8, chunk_steps=7)
    try:
        ids = [nd.nd_server_submit(s, p, y0, dt, steps) for p, y0, dt, steps, _ in cs]
        drain(nd, s)
        for rid, (p, y0, dt, steps, _) in zip(ids, cs):
            y = np.empty_like(y0)
            nd.nd_server_result(s, rid, y)
            if p.topo == nd.ND_RING:
                net = O.ring(O.KURAMOTO if p.model == 0 else O.FHN, p.n, p.radius, list(p.params)[:4])
            else:
                net = O.cube(12, 2, [0.0, 1.0, 0.8])
            ref, _, _ = O.run(net, y0, dt, steps)
            assert np.max(np.abs(y - ref)) / np.max(np.abs(ref)) < 1e-12
    finally:
        nd.nd_server_destroy(s)


def test_budget_is_respected_and_all_finish(nd):
    cs = cases(nd)
    fps = [nd.nd_footprint(c[0]) for c in cs]
    budget = 2 * max(fps) + 4096
    s = nd.nd_server_create(budget, max_slots=3, chunk_steps=32)
    try:
        ids = [nd.nd_server_submit(s, p, y0, dt, steps) for p, y0, dt, steps, _ in cs]
        for _ in range(10000):
            pending = nd.nd_server_pump(s)
            st = nd.nd_server_stats(s)
            assert st.bytes_in_use <= budget and st.running <= 3
            if pending == 0:
                break
        assert all(nd.nd_server_info(s, i).state == nd.ND_REQ_DONE for i in ids)
    finally:
        nd.nd_server_destroy(s)


def test_cancel_running_request_frees_its_slot(nd):
    p = nd.problem(nd.ND_FHN, nd.ND_RING, 4096, FHN_PRM, radius=1433)
    s = nd.nd_server_create(1 << 30, max_slots=1, chunk_steps=8)
    try:
        a = nd.nd_server_submit(s, p, inputs.fhn_circle(1, 4096), 0.01, 10000)
        b = nd.nd_server_submit(s, p, inputs.fhn_circle(2, 4096), 0.01, 16)
        nd.nd_server_pump(s)
        assert nd.nd_server_info(s, a).state == nd.ND_REQ_RUNNING
        assert nd.nd_server_info(s, b).state == nd.ND_REQ_QUEUED
        nd.nd_server_cancel(s, a)
        drain(nd, s)
        assert nd.nd_server_info(s, a).state == nd.ND_REQ_CANCELLED
        assert nd.nd_server_info(s, b).state == nd.ND_REQ_DONE
        assert nd.nd_server_stats(s).bytes_in_use == 0
    finally:
        nd.nd_server_destroy(s)


@pytest.mark.parametrize("grid", [0, 64])
def test_hh_requests_of_all_degrees_and_sizes(nd, grid):
    """HH requests join and leave one class while its chunks change shape (edges in
    flight, rows per work item, LDS): every result has the bits of its run alone."""
    shapes = [(3000, 5, 60), (700, 100, 25), (66000, 20, 40), (2500, 60, 30), (1500, 10, 90)]
    cs = []
    for n, deg, steps in shapes:
        rp, col, w = inputs.random_out_graph(deg, n, deg)
        cs.append((nd.problem(nd.ND_HH, nd.ND_CSR, n, HH_PRM, row_ptr=rp, col=col, weight=w,
                              per_elem=inputs.hh_iapp(9, n)), inputs.hh_state(9, n), steps))
    alone = [nd.simulate(p, y0, 0.01, steps)[0] for p, y0, steps in cs]
    print(f"case serve hh mix grid={grid}", flush=True)
    s = nd.nd_server_create(8 << 30, max_slots=3, chunk_steps=8, grid=grid)
    try:
        ids = []
        for p, y0, steps in cs:
            ids.append(nd.nd_server_submit(s, p, y0, 0.01, steps))
            nd.nd_server_pump(s)
        drain(nd, s)
        for rid, ya, (_, y0, _) in zip(ids, alone, cs):
            y = np.empty_like(y0)
            nd.nd_server_result(s, rid, y)
            assert np.array_equal(y, ya)
    finally:
        nd.nd_server_destroy(s)
