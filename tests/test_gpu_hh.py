"""GPU parity of the Hodgkin-Huxley CSR path against the FP64 CPU oracle,
through the C ABI."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2410_19075_amd import inputs

pytestmark = pytest.mark.gpu

HH_PRM = [1.0, 120.0, 36.0, 0.3, 50.0, -77.0, -54.387, 0.0, 0.0, 2.0]


@pytest.fixture(scope="module")
def nd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_19075_amd import nd as _nd
    return _nd


def normwise(a, ref):
    a = a.reshape(4, -1)
    ref = ref.reshape(4, -1)
    return max(np.max(np.abs(a[v] - ref[v])) / np.max(np.abs(ref[v])) for v in range(4))


def hh_case(nd, n, deg, seed, steps, prec=0, cfg=None, dt=0.01):
    rp, col, w = inputs.random_out_graph(seed, n, deg)
    iapp = inputs.hh_iapp(seed, n)
    y0 = inputs.hh_state(seed, n)
    p = nd.problem(nd.ND_HH, nd.ND_CSR, n, HH_PRM, precision=prec, row_ptr=rp, col=col, weight=w, per_elem=iapp)
    h = nd.nd_create(p)
    try:
        if cfg:
            c = nd.nd_get_config(h)
            for k, v in cfg.items():
                setattr(c, k, v)
            nd.nd_set_config(h, c)
        nd.nd_set_state(h, y0, on_device=0)
        nd.nd_run(h, dt, steps)
        y = np.empty_like(y0)
        nd.nd_get_state(h, y, on_device=0)
    finally:
        nd.nd_destroy(h)
    ref, _, _ = O.run(O.csr(n, rp, col, w, HH_PRM, iapp), y0, dt, steps)
    return y, ref


@pytest.mark.parametrize("n,deg,steps", [(50, 7, 300), (2000, 50, 200), (1000, 999 // 10, 100), (777, 1, 50)])
def test_hh_fp64_parity(nd, n, deg, steps):
    print(f"case hh n={n} deg={deg}", flush=True)
    y, ref = hh_case(nd, n, deg, n + deg, steps)
    assert normwise(y, ref) < 1e-12


@pytest.mark.parametrize("ept", [2, 4, 8, 16])
def test_hh_edges_per_thread(nd, ept):
    print(f"case hh ept={ept}", flush=True)
    y, ref = hh_case(nd, 3000, 100, 5, 20, cfg=dict(tile_y=ept))
    assert normwise(y, ref) < 1e-12


def test_hh_edges_per_thread_bitwise(nd):
    """Every row's products are added in edge order whatever the chunking, so the
    result does not depend on the edges-per-thread setting at all."""
    ys = [hh_case(nd, 2500, 60, 9, 10, cfg=dict(tile_y=e))[0] for e in (2, 4, 8, 16)]
    for y in ys[1:]:
        assert np.array_equal(y, ys[0])


def hub_graph(n, deg, hub, empty, seed):
    """Random out-degree `deg` graph plus every node feeding `hub`, with the rows
    in `empty` stripped of all in-edges; CSR by target, sources ascending."""
    rng = np.random.default_rng(seed)
    src = np.repeat(np.arange(n), deg)
    dst = rng.integers(0, n, size=src.size)
    keep = dst != src
    src, dst = src[keep], dst[keep]
    src = np.concatenate([src, np.delete(np.arange(n), hub)])
    dst = np.concatenate([dst, np.full(n - 1, hub)])
    keep = ~np.isin(dst, empty)
    src, dst = src[keep], dst[keep]
    order = np.lexsort((src, dst))
    src, dst = src[order], dst[order]
    rp = np.zeros(n + 1, dtype=np.int64)
    rp[1:] = np.cumsum(np.bincount(dst, minlength=n))
    w = rng.uniform(0.0, 0.1, size=src.size)
    return rp, src.astype(np.int32), w


@pytest.mark.parametrize("ept", [2, 16])
def test_hh_hub_row_spans_chunks(nd, ept):
    """A row whose in-edges of one source block exceed a whole chunk (hub with
    in-degree n-1, ~5000 edges per block), and rows with no in-edges at all."""
    n = 40000
    rp, col, w = hub_graph(n, 3, 7, np.arange(100, 300), 11)
    assert np.diff(rp)[100:300].max() == 0 and np.diff(rp)[7] >= n - 1
    iapp = inputs.hh_iapp(11, n)
    y0 = inputs.hh_state(11, n)
    p = nd.problem(nd.ND_HH, nd.ND_CSR, n, HH_PRM, row_ptr=rp, col=col, weight=w, per_elem=iapp)
    h = nd.nd_create(p)
    try:
        c = nd.nd_get_config(h)
        c.tile_y = ept
        nd.nd_set_config(h, c)
        nd.nd_set_state(h, y0, on_device=0)
        nd.nd_run(h, 0.01, 5)
        y = np.empty_like(y0)
        nd.nd_get_state(h, y, on_device=0)
    finally:
        nd.nd_destroy(h)
    ref, _, _ = O.run(O.csr(n, rp, col, w, HH_PRM, iapp), y0, 0.01, 5)
    assert normwise(y, ref) < 1e-12


def test_hh_persistent_grid_and_chunks(nd):
    y, ref = hh_case(nd, 5000, 30, 6, 45, cfg=dict(grid=8, chunk=7))
    assert normwise(y, ref) < 1e-12


def test_hh_large_graph_few_steps(nd):
    """10^5 neurons with out-degree 100 (10^7 synapses)."""
    y, ref = hh_case(nd, 100000, 100, 7, 3)
    assert normwise(y, ref) < 1e-12


def test_hh_fp32_bulk(nd):
    y, ref = hh_case(nd, 2000, 50, 8, 200, prec=1)
    e = normwise(y, ref)
    print(f"hh fp32 error {e:.3e}")
    assert e < 1e-4


def test_hh_fp32_bulk_1e5_deg100_200_steps(nd):
    """FP32-bulk over the 200-step horizon at the benchmark's out-degree (10^5
    neurons, 10^7 synapses; the launch configuration of the 10^6 network:
    source blocks per XCD, 256 rows per work item, 8 edges per thread)
    against the oracle."""
    print("case hh 1e5 x 100 fp32-bulk, 200 steps", flush=True)
    y, ref = hh_case(nd, 100000, 100, 9, 200, prec=1)
    e = normwise(y, ref)
    print(f"hh 1e5 fp32-bulk 200-step error {e:.3e}")
    assert e < 1e-4


@pytest.fixture(scope="module")
def hh_full():
    """The benchmark's network (10^6 neurons, out-degree 100) and the oracle's
    state after two steps, shared by the FP64 and FP32-bulk full-size tests."""
    n, deg, seed = 1000000, 100, 1
    rp, col, w = inputs.random_out_graph(seed, n, deg)
    iapp = inputs.hh_iapp(seed, n)
    y0 = inputs.hh_state(seed, n)
    ref, _, _ = O.run(O.csr(n, rp, col, w, HH_PRM, iapp), y0, 0.01, 2)
    return n, rp, col, w, iapp, y0, ref


def hh_run(nd, net, prec, steps):
    n, rp, col, w, iapp, y0, _ = net
    p = nd.problem(nd.ND_HH, nd.ND_CSR, n, HH_PRM, precision=prec, row_ptr=rp, col=col, weight=w, per_elem=iapp)
    y, _, _ = nd.simulate(p, y0, 0.01, steps)
    return y


def test_hh_full_size_two_steps(nd, hh_full):
    """The benchmark's workload at full size and in its launch configuration:
    10^6 neurons, out-degree 100 (10^8 synapses), two steps against the oracle."""
    print("case full HH 1e6 x 100, two steps", flush=True)
    assert normwise(hh_run(nd, hh_full, 0, 2), hh_full[-1]) < 1e-12


def test_hh_full_size_fp32_bulk_two_steps(nd, hh_full):
    """FP32-bulk at full size (FP32 weights and activations, FP64 synaptic sums
    and state), two steps against the oracle."""
    print("case full HH 1e6 x 100 fp32-bulk, two steps", flush=True)
    e = normwise(hh_run(nd, hh_full, 1, 2), hh_full[-1])
    print(f"hh 1e6 fp32-bulk two-step error {e:.3e}")
    assert e < 1e-4


def test_hh_full_size_fp32_bulk_200_steps_against_fp64(nd, hh_full):
    """FP32-bulk at full size over the 200-step horizon against the FP64 path,
    which the two-step oracle test holds at this size."""
    print("case full HH 1e6 x 100 fp32-bulk vs fp64, 200 steps", flush=True)
    e = normwise(hh_run(nd, hh_full, 1, 200), hh_run(nd, hh_full, 0, 200))
    print(f"hh 1e6 fp32-bulk vs fp64 after 200 steps {e:.3e}")
    assert e < 1e-4


def run_net(nd, n, graph, steps, prec=0, seed=3):
    rp, col, w = graph
    iapp, y0 = inputs.hh_iapp(seed, n), inputs.hh_state(seed, n)
    p = nd.problem(nd.ND_HH, nd.ND_CSR, n, HH_PRM, precision=prec, row_ptr=rp, col=col, weight=w, per_elem=iapp)
    y, _, _ = nd.simulate(p, y0, 0.01, steps)
    return y, p, y0, iapp


def test_hh_hub_row_spans_sorted_chunks(nd):
    """A row with more in-edges of one source block (10^4) than a chunk holds: its
    products are added over two chunks of sorted edges.  1e-12 as for every FP64
    run of a few steps: each row's products are added in edge order."""
    n = 80000
    g = hub_graph(n, 2, 7, np.arange(600, 700), 12)
    print("case hh hub over sorted chunks", flush=True)
    y, _, y0, iapp = run_net(nd, n, g, 3)
    ref, _, _ = O.run(O.csr(n, *g, HH_PRM, iapp), y0, 0.01, 3)
    assert normwise(y, ref) < 1e-12


def test_hh_rows_in_any_order(nd):
    """Rows whose sources are not ascending: the sums take the given order inside a
    source block, so two orders of the same rows agree to rounding (1e-13)."""
    n, deg = 5000, 40
    rp, col, w = inputs.random_out_graph(4, n, deg)
    rng = np.random.default_rng(4)
    order = np.lexsort((rng.random(col.size), np.repeat(np.arange(n), np.diff(rp))))
    print("case hh rows in any order", flush=True)
    a = run_net(nd, n, (rp, col, w), 5)[0]
    b = run_net(nd, n, (rp, col[order].copy(), w[order].copy()), 5)[0]
    assert normwise(b, a) < 1e-13


@pytest.mark.parametrize("extra", [0, 1])
def test_hh_largest_packed_and_first_unpacked_size(nd, extra):
    """2^22 neurons, the most whose edges pack a source and a slot into one word,
    and one more, which keeps plain sources: in-edges from both ends of every
    source block, one step against the oracle."""
    n = (1 << 22) + extra
    i = np.arange(n, dtype=np.int64)
    block = (i * 2654435761) % 8
    first = (block * n + 7) // 8
    last = ((block + 1) * n + 7) // 8 - 1
    col = np.stack([first, last], 1).astype(np.int32).ravel()
    rp = 2 * np.arange(n + 1, dtype=np.int64)
    w = inputs.uniform(6, inputs.TAG_WEIGHT, 2 * n) * 0.1
    print(f"case hh n={n}", flush=True)
    y, _, y0, iapp = run_net(nd, n, (rp, col, w), 1)
    ref, _, _ = O.run(O.csr(n, rp, col, w, HH_PRM, iapp), y0, 0.01, 1)
    assert normwise(y, ref) < 1e-12


def test_hh_batch_of_mixed_sizes_and_degrees(nd):
    """Networks with 256 and 512 rows per work item and every default of edges per
    thread in one batch call: the same bits as alone."""
    cases = [(700, 5), (3000, 100), (70000, 3), (66000, 40), (1500, 90)]
    print("case hh mixed batch", flush=True)
    alone, hs, y0s = [], [], []
    try:
        for n, deg in cases:
            y, p, y0, _ = run_net(nd, n, inputs.random_out_graph(deg, n, deg), 4)
            alone.append(y)
            y0s.append(y0)
            hs.append(nd.nd_create(p))
        for h, y0 in zip(hs, y0s):
            nd.nd_set_state(h, y0, on_device=0)
        nd.nd_run_batch(hs, [0.01] * len(hs), [4] * len(hs))
        for h, y in zip(hs, alone):
            got = np.empty_like(y)
            nd.nd_get_state(h, got, on_device=0)
            assert np.array_equal(got, y)
    finally:
        for h in hs:
            nd.nd_destroy(h)


@pytest.mark.parametrize("n", [3000, 70001])
@pytest.mark.parametrize("prec", [0, 1])
def test_hh_banded_graph_on_a_small_grid(nd, n, prec):
    """Rows with sources within 10 places, every 64th without any: nearly all (row
    tile, source block) items have no edges.  Eight workgroups that take many items
    each give the bits of one workgroup per item; FP64 also against the oracle."""
    rng = np.random.default_rng(n)
    deg = np.where(np.arange(n) % 64 == 0, 0, 6)
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    off = np.array([-10, -4, -1, 2, 3, 10])
    col = ((np.arange(n)[deg > 0, None] + off[None, :]) % n).astype(np.int32).ravel()
    w = rng.random(col.size) * 0.1
    iapp, y0 = inputs.hh_iapp(3, n), inputs.hh_state(3, n)
    p = nd.problem(nd.ND_HH, nd.ND_CSR, n, HH_PRM, precision=prec, row_ptr=rp, col=col, weight=w, per_elem=iapp)
    got = []
    for grid in (0, 8):
        print(f"case hh banded n={n} prec={prec} grid={grid}", flush=True)
        h = nd.nd_create(p)
        try:
            c = nd.nd_get_config(h)
            c.grid = grid
            nd.nd_set_config(h, c)
            nd.nd_set_state(h, y0, on_device=0)
            nd.nd_run(h, 0.01, 5)
            y = np.empty_like(y0)
            nd.nd_get_state(h, y, on_device=0)
            got.append(y)
        finally:
            nd.nd_destroy(h)
    assert np.array_equal(got[0], got[1])
    if prec == 0:
        ref, _, _ = O.run(O.csr(n, rp, col, w, HH_PRM, iapp), y0, 0.01, 5)
        assert normwise(got[0], ref) < 1e-12


def graph_nodes(torch, g):
    """Number of nodes of a captured (kept) graph."""
    import ctypes
    import os
    hip = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("prec", [0, 1])
def test_hh_networks_of_all_degrees_and_sizes_share_launches(nd, prec):
    """A batch of networks with every default of edges per thread takes as many
    launches as one of equal networks, with both row counts per work item one more
    per stage, and gives each network the bits of its run alone; so does an explicit
    value beside others."""
    import torch
    steps = 4
    cases = {"equal": [(700, 5)] * 4, "degrees": [(700, 5), (900, 40), (3000, 100), (1500, 60)],
             "sizes": [(700, 5), (66000, 40), (3000, 100), (1500, 60)]}
    st = torch.cuda.Stream()
    nodes = {}
    for kind, shapes in cases.items():
        hs, y0s, alone = [], [], []
        try:
            for n, deg in shapes:
                rp, col, w = inputs.random_out_graph(deg, n, deg)
                y0s.append(torch.from_numpy(inputs.hh_state(3, n)).cuda())
                hs.append(nd.nd_create(nd.problem(nd.ND_HH, nd.ND_CSR, n, HH_PRM, precision=prec, row_ptr=rp, col=col,
                                                  weight=w, per_elem=inputs.hh_iapp(3, n))))
            c = nd.nd_get_config(hs[-1])
            c.tile_y = 2
            nd.nd_set_config(hs[-1], c)
            print(f"case hh shared launches {kind} prec={prec}", flush=True)
            with torch.cuda.stream(st):
                for h, y0 in zip(hs, y0s):
                    nd.nd_set_state(h, y0, stream=st)
                    nd.nd_run(h, 0.01, steps, stream=st)
                    alone.append(torch.empty_like(y0))
                    nd.nd_get_state(h, alone[-1], stream=st)
                    nd.nd_set_state(h, y0, stream=st)
                nd.nd_run_batch_noalloc(hs, [0.01] * len(hs), [steps] * len(hs), stream=st)
                for h, y in zip(hs, alone):
                    got = torch.empty_like(y)
                    nd.nd_get_state(h, got, stream=st)
                    nd.nd_sync(h, stream=st)
                    assert torch.equal(got, y)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph(keep_graph=True)
            with torch.cuda.graph(g, stream=st):
                nd.nd_run_batch_noalloc(hs, [0.01] * len(hs), [steps] * len(hs), stream=st)
            nodes[kind] = graph_nodes(torch, g)
        finally:
            for h in hs:
                nd.nd_destroy(h)
    assert nodes["equal"] == nodes["degrees"] == nodes["sizes"] - 4 * steps, nodes


@pytest.mark.parametrize("n, rows", [(65535, 256), (65536, 512)])
def test_hh_config_reports_the_rows_that_run(nd, n, rows):
    """nd_get_config gives the rows per work item of the size; set back, or with the
    256 that configurations of every size held before, it is accepted and changes
    nothing, other values are refused."""
    g = inputs.random_out_graph(8, n, 4)
    y, p, y0, _ = run_net(nd, n, g, 2)
    h = nd.nd_create(p)
    try:
        c = nd.nd_get_config(h)
        assert (c.tile, c.block) == (rows, rows)
        for tile in (rows, 256):
            print(f"case hh config n={n} tile={tile}", flush=True)
            c.tile = tile
            nd.nd_set_config(h, c)
            c = nd.nd_get_config(h)
            assert (c.tile, c.block) == (rows, rows)
            nd.nd_set_state(h, y0, on_device=0)
            nd.nd_run(h, 0.01, 2)
            got = np.empty_like(y)
            nd.nd_get_state(h, got, on_device=0)
            assert np.array_equal(got, y)
        for tile in (0, 128, 2 * rows):
            c.tile = tile
            with pytest.raises(nd.NDError):
                nd.nd_set_config(h, c)
    finally:
        nd.nd_destroy(h)


def test_hh_batch_of_both_sizes_beyond_the_cache(nd):
    """Networks of both row counts whose edges together exceed what shares launches
    (192 MB): each has the bits of its run alone, in both kinds of batch run."""
    shapes = [(30000, 120), (70000, 200), (500, 30)]
    rng = np.random.default_rng(5)
    hs, y0s, alone = [], [], []
    print("case hh batch beyond the cache", flush=True)
    try:
        for n, deg in shapes:
            g = (np.arange(n + 1, dtype=np.int64) * deg,
                 np.sort(rng.integers(0, n, size=(n, deg), dtype=np.int32), axis=1).ravel(), rng.random(n * deg) * 0.1)
            y, p, y0, _ = run_net(nd, n, g, 3)
            alone.append(y)
            y0s.append(y0)
            hs.append(nd.nd_create(p))
        for run in (nd.nd_run_batch, nd.nd_run_batch_noalloc):
            for h, y0 in zip(hs, y0s):
                nd.nd_set_state(h, y0, on_device=0)
            run(hs, [0.01] * len(hs), [3] * len(hs))
            for h, y in zip(hs, alone):
                got = np.empty_like(y)
                nd.nd_get_state(h, got, on_device=0)
                assert np.array_equal(got, y)
    finally:
        for h in hs:
            nd.nd_destroy(h)
