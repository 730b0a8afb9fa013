"""k nearest neighbours and the top-k merge on the GPU against the fp64-free
oracle (fp32 distances, exact order): bit-exact indices and distances (GPU)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import log

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def gpu_knn(x_q, x_c, k, c_index0=0, q_self0=-1, group_q=None, group_c=None, mode=0, with_d2=True):
    import torch
    import paper_2607_05439_amd as dcp
    xq, xc = dev(x_q), dev(x_c)
    gq = None if group_q is None else dev(group_q)
    gc = None if group_c is None else dev(group_c)
    n_q = len(x_q)
    idx = torch.full((max(n_q, 1), k), -7, dtype=torch.int32, device="cuda:0")
    d2 = torch.full((max(n_q, 1), k), -7.0, dtype=torch.float32, device="cuda:0") if with_d2 else None
    ws_bytes = dcp.dcp_knn_workspace_size(len(x_c))
    ws = torch.full((max(ws_bytes, 1),), 0xA5, dtype=torch.uint8, device="cuda:0")  # stale contents
    dcp.dcp_knn_topk(xq, n_q, xc, len(x_c), c_index0, q_self0, gq, gc, mode, k, idx, d2, ws, ws_bytes)
    return idx.cpu().numpy()[:n_q], (d2.cpu().numpy()[:n_q] if with_d2 else None)


def same(got, ref, what):
    gi, gd = got
    ri, rd = ref
    bad = np.flatnonzero((gi != ri).any(1) | ((gd != rd).any(1) if gd is not None else False))
    if len(bad):
        r = bad[0]
        log(f"  {what}: {len(bad)} rows differ; row {r}: got {gi[r][:8]} ref {ri[r][:8]}")
    assert len(bad) == 0, what


@pytest.mark.parametrize("name", ["knn300", "knn5000"])
def test_whole_workload_bit_exact(name):
    wl = synth.KNN_WORKLOADS[name]
    x = synth.coords(wl)
    q = x[wl.q_row0:wl.q_row0 + wl.n_q]
    ref = oracle.knn(q, x, wl.k)
    log(f"case {name} k={wl.k}: self order and plain order")
    same(gpu_knn(q, x, wl.k, q_self0=wl.q_row0), ref, "self-start")
    same(gpu_knn(q, x, wl.k), ref, "index order")


@pytest.mark.parametrize("k", [1, 63, 64, 65, 200, 256])
def test_k_values(k):
    wl = synth.KNN_WORKLOADS["knn5000"]
    x = synth.coords(wl)
    q = x[1000:1700]
    same(gpu_knn(q, x, k, q_self0=1000), oracle.knn(q, x, k), f"k={k}")


def test_group_modes():
    wl = synth.KNN_WORKLOADS["knn5000"]
    x = synth.coords(wl)
    g = synth.chain_ids(wl)
    rows = np.arange(0, 5000, 3)
    for mode in (1, 2):
        ref = oracle.knn(x[rows], x, 128, group_q=g[rows], group_c=g, group_mode=mode)
        got = gpu_knn(x[rows], x, 128, group_q=g[rows], group_c=g, mode=mode)
        same(got, ref, f"group mode {mode}")
        if mode == 2:
            assert ((got[0] // wl.per_chain) != (rows // wl.per_chain)[:, None]).all()


def test_ring_blocks_and_merge():
    """Per-block top-k of the candidate blocks (chunk rule), merged in ring
    order on the GPU, equals the one-call result."""
    import torch
    import paper_2607_05439_amd as dcp
    wl = synth.KNN_WORKLOADS["knn5000"]
    x = synth.coords(wl)
    q = x[2000:2600]
    k = 128
    full = gpu_knn(q, x, k)
    run_i = dev(np.full((len(q), k), -1, dtype=np.int32))
    run_d = dev(np.full((len(q), k), np.inf, dtype=np.float32))
    for b in range(5):
        size, start = oracle.chunk(len(x), 5, b)
        bi, bd = gpu_knn(q, x[start:start + size], k, c_index0=start)
        out_i = torch.empty_like(run_i)
        out_d = torch.empty_like(run_d)
        dcp.dcp_topk_merge(len(q), k, run_i, run_d, dev(bi), dev(bd), out_i, out_d)
        run_i, run_d = out_i, out_d
    same((run_i.cpu().numpy(), run_d.cpu().numpy()), full, "ring merge")
    same(full, oracle.knn(q, x, k, n_blocks=5), "oracle ring form")


def test_topk_merge_matches_oracle():
    import torch
    import paper_2607_05439_amd as dcp
    r = np.random.default_rng(5)
    for k in (16, 128, 256):
        n = 300
        lists = []
        for _ in range(2):
            d = np.sort(r.integers(0, 50, (n, k)).astype(np.float32), axis=1)  # many equal distances
            i = r.integers(0, 10000, (n, k)).astype(np.int32)
            o = np.lexsort((i, d), axis=1)
            d, i = np.take_along_axis(d, o, 1), np.take_along_axis(i, o, 1)
            cut = r.integers(0, k + 1, n)  # ragged: empty tails
            for row in range(n):
                i[row, cut[row]:] = -1
                d[row, cut[row]:] = np.inf
            lists.append((i, d))
        (ia, da), (ib, db) = lists
        ref = oracle.topk_merge(ia, da, ib, db)
        oi = torch.empty((n, k), dtype=torch.int32, device="cuda:0")
        od = torch.empty((n, k), dtype=torch.float32, device="cuda:0")
        dcp.dcp_topk_merge(n, k, dev(ia), dev(da), dev(ib), dev(db), oi, od)
        # equal (d2, index) pairs may come from either list: compare the pairs
        same((oi.cpu().numpy(), od.cpu().numpy()), ref, f"merge k={k}")


def test_ties_on_a_grid_and_duplicates():
    """Integer coordinates on a 9x9x9 grid: every point repeats about four
    times and most distances tie, so the order rests on the index rule."""
    r = np.random.default_rng(11)
    x = r.integers(-4, 5, (3000, 3)).astype(np.float32)
    for k in (1, 100, 256):
        same(gpu_knn(x[:333], x, k, q_self0=0), oracle.knn(x[:333], x, k), f"grid k={k}")
    same(gpu_knn(x[1:2], x, 7), oracle.knn(x[1:2], x, 7), "one query")


@pytest.mark.parametrize("scale,shift", [(1.0, 3000.0), (1.0, -250000.0), (1e-4, 0.0), (1e-4, 7.0), (1e5, 0.0)])
def test_coordinate_magnitudes(scale, shift):
    """The candidate prefilter bounds |c|^2 - 2 c.q with a rounding margin
    that grows with |q|: structures far from the origin (where most of that
    expression cancels), at sub-angstrom scales and at very large scales give
    the same exact lists as the oracle."""
    x0 = synth.coords(synth.KNN_WORKLOADS["knn5000"])
    x = (x0.astype(np.float64) * scale + shift).astype(np.float32)
    q = x[2000:2600]
    log(f"case scale={scale} shift={shift}")
    for k in (1, 128):
        same(gpu_knn(q, x, k, q_self0=2000), oracle.knn(q, x, k), f"scale={scale} shift={shift} k={k}")


def test_short_and_empty_candidate_sets():
    x = synth.coords(synth.KNN_WORKLOADS["knn300"])
    same(gpu_knn(x[:40], x[:30], 64), oracle.knn(x[:40], x[:30], 64), "fewer candidates than k")
    gi, gd = gpu_knn(x[:5], x[:0], 8)
    assert (gi == -1).all() and np.isinf(gd).all()
    gi, gd = gpu_knn(x[:5], x, 8, with_d2=False)
    assert np.array_equal(gi, oracle.knn(x[:5], x, 8)[0])


def test_knn96k_sampled_rows_and_ring_form():
    """Full size: the 24000-atom query stripe of the 96000-atom assembly in the
    benchmark's call (one call over all candidates), checked bit-exact on
    sampled rows; the 4-block ring form gives identical lists."""
    import torch
    import paper_2607_05439_amd as dcp
    wl = synth.KNN_WORKLOADS["knn96k"]
    x = synth.coords(wl)
    q = x[wl.q_row0:wl.q_row0 + wl.n_q]
    log("case knn96k: one call, k=128")
    gi, gd = gpu_knn(q, x, wl.k, q_self0=wl.q_row0)
    rows = {0, wl.n_q - 1}
    for b in range(wl.n_col_blocks):
        size, start = oracle.chunk(wl.n_atoms, wl.n_col_blocks, b)
        for atom in (start - 1, start, start + size - 1):
            if wl.q_row0 <= atom < wl.q_row0 + wl.n_q:
                rows.add(atom - wl.q_row0)
    rows.update(int(v) for v in np.random.default_rng(0).choice(wl.n_q, 200, replace=False))
    rows = sorted(rows)
    same((gi[rows], gd[rows]), oracle.knn(q[rows], x, wl.k), "sampled rows")
    log("case knn96k: 4-block ring form")
    run_i = dev(np.full((wl.n_q, wl.k), -1, dtype=np.int32))
    run_d = dev(np.full((wl.n_q, wl.k), np.inf, dtype=np.float32))
    for b in range(wl.n_col_blocks):
        size, start = oracle.chunk(wl.n_atoms, wl.n_col_blocks, b)
        bi, bd = gpu_knn(q, x[start:start + size], wl.k, c_index0=start,
                         q_self0=wl.q_row0 - start if start <= wl.q_row0 < start + size else -1)
        oi, od = torch.empty_like(run_i), torch.empty_like(run_d)
        dcp.dcp_topk_merge(wl.n_q, wl.k, run_i, run_d, dev(bi), dev(bd), oi, od)
        run_i, run_d = oi, od
    same((run_i.cpu().numpy(), run_d.cpu().numpy()), (gi, gd), "ring form")


@pytest.mark.parametrize("k,lattice,mode", [(1, False, 0), (64, False, 0), (100, True, 0), (128, False, 0),
                                            (200, False, 0), (256, True, 0), (100, True, 1), (200, False, 1)])
def test_two_queries_per_wave(k, lattice, mode):
    """More than 16384 queries run two per wave: whole lists against the same queries in stripes that
    run one per wave, and sampled rows against the oracle; an odd query count, a last step of a
    few candidates, and (lattice) distances that tie in every list."""
    r = np.random.default_rng(k)
    n_q, n_c = 16387, 2311
    x = (r.integers(0, 9, (n_c, 3)) if lattice else 40.0 * r.standard_normal((n_c, 3))).astype(np.float32)
    q = (r.integers(0, 9, (n_q, 3)) if lattice else 40.0 * r.standard_normal((n_q, 3))).astype(np.float32)
    q[:n_c] = x  # the first queries are the candidates
    g = (np.arange(n_q) % n_c // 400).astype(np.int32)
    gq, gc = (g, g[:n_c]) if mode else (None, None)
    got = gpu_knn(q, x, k, 5, 0, gq, gc, mode)
    a = gpu_knn(q[:9000], x, k, 5, 0, gq if gq is None else gq[:9000], gc, mode)
    b = gpu_knn(q[9000:], x, k, 5, -1, gq if gq is None else gq[9000:], gc, mode)
    same(got, (np.concatenate([a[0], b[0]]), np.concatenate([a[1], b[1]])), "two per wave against one")
    rows = np.concatenate([np.arange(0, n_q, 97), [n_q - 2, n_q - 1]])
    ri, rd = oracle.knn(q[rows], x, k, group_q=None if gq is None else gq[rows], group_c=gc, group_mode=mode)
    same((got[0][rows], got[1][rows]), (np.where(ri < 0, ri, ri + 5), rd), "against the oracle")


@pytest.mark.parametrize("k", [3, 200])
def test_coordinates_beyond_half_the_largest_float(k):
    """Coordinates whose double is infinite in fp32: differences of such neighbours are ordinary
    numbers (or 0 at the same point), and squares of the others overflow to +inf, which ties."""
    x = np.random.default_rng(k).standard_normal((300, 3)).astype(np.float32)
    x[100:] *= np.float32(0.7e38)  # up to about 2.4e38, half of them beyond 1.7e38 in some coordinate
    x[[7, 8, 290]] = 2e38
    x[9], x[291] = np.float32(3.4e38), np.float32(-3.4e38)
    got = gpu_knn(x, x, k, q_self0=0)
    assert got[0][7][:3].tolist() == [7, 8, 290] and (got[1][7][:3] == 0).all()
    same(got, oracle.knn(x, x, k), "beyond half the largest float")


@pytest.mark.parametrize("k", [1, 64, 100, 128, 200, 256])
def test_shared_kth_distances(k):
    """Padding atoms at one point, a coarse lattice and both: the k-th distance is shared by more
    candidates than the list holds, and the smaller indices win, up to the largest index there is."""
    r = np.random.default_rng(k)
    pad = np.zeros((700, 3), np.float32)
    grid = r.integers(0, 4, (700, 3)).astype(np.float32)
    for x, index0 in ((pad, 0), (grid, 2**31 - 1 - 700), (np.concatenate([grid, pad, grid[::-1]]), 12345)):
        ri, rd = oracle.knn(x, x, k)
        got = gpu_knn(x, x, k, c_index0=index0, q_self0=0)
        same(got, (np.where(ri < 0, ri, ri + index0), rd), f"{len(x)} candidates from index {index0}")


def test_shared_distances_take_no_longer():
    """Atoms at one point enter a full list no more often than atoms in general position: a candidate
    at the k-th distance with a larger index is turned away before the selection (when it was not,
    these calls took five times as long as the others; the bound is twice)."""
    import torch
    import paper_2607_05439_amd as dcp
    n, k = 4800, 128
    ws_bytes = dcp.dcp_knn_workspace_size(n)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda:0")
    idx = torch.empty((n, k), dtype=torch.int32, device="cuda:0")

    def us(x):
        best = float("inf")
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            dcp.dcp_knn_topk(x, n, x, n, 0, 0, None, None, 0, k, idx, None, ws, ws_bytes)
            b.record()
            torch.cuda.synchronize()
            best = min(best, 1e3 * a.elapsed_time(b))
        return best

    one, spread = us(torch.zeros((n, 3), device="cuda:0")), us(30 * torch.randn((n, 3), device="cuda:0"))
    log(f"case {n} atoms, k = {k}: at one point {one:.1f} us, in general position {spread:.1f} us")
    assert one <= 2 * spread
