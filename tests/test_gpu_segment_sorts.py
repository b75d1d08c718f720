"""The two sorts of a segment table (ensembles of unequal lengths): by
splitters and by radix passes, which a batch takes for ensembles above 2^20 +
2^16 keys and where its timing prefers them.  Both against numpy's stable sort
through the library's internal entries, and a batch that holds both kinds."""
import ctypes

import numpy as np
import pytest

import paper_1912_09240_amd as pr
from oracle import restrict as OR

pytestmark = pytest.mark.gpu

LONGEST = 2 ** 20 + 2 ** 16  # keys of an ensemble that goes by splitters


class _Layout(ctypes.Structure):  # pr::SortLayout
    _fields_ = [("n", ctypes.c_int64), ("nblk", ctypes.c_int), ("nseg", ctypes.c_int), ("segs", ctypes.c_void_p),
                ("tile_seg", ctypes.c_void_p), ("guard", ctypes.c_void_p), ("max_n", ctypes.c_int64),
                ("radix", ctypes.c_bool)]


SEG = np.dtype([("base", "<i8"), ("n", "<i8"), ("tile0", "<i8"), ("nblk", "<i4"), ("qrow", "<i4")])  # pr::SortSeg


def _entries():
    lib = ctypes.CDLL(pr.lib()._name)
    sort = lib["_ZN2pr17restrict_segmentsEPKdRKNS_10SortLayoutElliPdPjPvP12ihipStream_t"]
    sort.argtypes = [ctypes.c_void_p, ctypes.POINTER(_Layout), ctypes.c_int64, ctypes.c_int64, ctypes.c_int,
                     ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
    size = lib["_ZN2pr13sort_ws_bytesElliib"]
    size.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_bool]
    size.restype = ctypes.c_size_t
    return sort, size


def _values(case, n, rng):
    x = rng.normal(0.0, 1.0, n)
    if case == "ties":  # runs of equal high halves too long for the fix-up: the complete sort
        x = np.round(x * 20.0) / 20.0
    elif case == "near":  # short runs that agree in the high half only
        x = 1.0 + (rng.integers(0, max(1, n // 8), n) * 2.0 ** -20) + rng.integers(0, 1000, n) * 2.0 ** -52
    return x


@pytest.mark.parametrize("case", ["smooth", "near", "ties"])
@pytest.mark.parametrize("radix", [False, True])
@pytest.mark.parametrize("sizes", [(1, 2, 4095, 4096, 4097, 7168, 7169), (65_536, 3000, 2 ** 20, 70_001),
                                   (LONGEST + 1, 1, 5000)])
def test_segment_table(sizes, radix, case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"segment table sizes={sizes} radix={radix} {case}", flush=True)
    sort, size = _entries()
    nq, rng = 50, np.random.default_rng(31)
    xs = [_values(case, n, rng) for n in sizes]
    segs, tile_seg, base = np.zeros(len(sizes), SEG), [], 0
    for i, n in enumerate(sizes):
        nblk = (n + 4095) // 4096
        segs[i] = (base, n, len(tile_seg), nblk, len(sizes) - 1 - i)
        tile_seg += [i] * nblk
        base += n
    total, tiles = base, len(tile_seg)
    x = torch.from_numpy(np.concatenate(xs)).cuda()
    d_segs = torch.from_numpy(segs.view(np.uint8)).cuda()
    d_tiles = torch.tensor(tile_seg, dtype=torch.int32, device="cuda")
    ws = torch.empty(size(total, tiles, len(sizes), pr.PR_F64, True), dtype=torch.uint8, device="cuda")
    q = torch.zeros((2, len(sizes), nq + 1), dtype=torch.float64, device="cuda")
    rank = torch.zeros(total, dtype=torch.int32, device="cuda")
    layout = _Layout(0, 0, len(sizes), d_segs.data_ptr(), d_tiles.data_ptr(), None, max(sizes), radix)
    st = torch.cuda.current_stream().cuda_stream
    for out, r in ((q[0], rank.data_ptr()), (q[1], None)):  # with ranks, and knots alone
        assert sort(x.data_ptr(), ctypes.byref(layout), total, tiles, nq, out.data_ptr(), r, ws.data_ptr(), st) == 0
    torch.cuda.synchronize()
    ranks = rank.cpu().numpy().view(np.uint32)
    assert torch.equal(q[0], q[1])
    for i, n in enumerate(sizes):
        _, want, srt = OR.sort_ranks(xs[i])
        b = int(segs[i]["base"])
        assert np.array_equal(ranks[b:b + n], want), n
        assert np.array_equal(q[0, len(sizes) - 1 - i].cpu().numpy(), OR.hazen_knots(srt, nq)), n


def test_batch_of_short_and_longest_ensembles():
    """One instance above the splitter sort's lengths (radix passes) beside
    ones below (splitters), sorted in turn in one workspace: every instance as
    its own handle computes it, bit for bit, in launches and in the graph."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sizes, ids = (4097, LONGEST + 4099, 70_001, 500), (3, 4, 5, 6)
    print(f"batch of short and longest ensembles {sizes}", flush=True)
    sde, sched, grid = pr.Sde(lam=1.1, eps=0.1), pr.Schedule(8, 2, 0.002), pr.Grid(n_cells=50, n_q=40)

    def states(get, n):
        out = []
        for t in range(3):
            b = [torch.empty(v, dtype=torch.float64, device="cuda") for v in (n, n, 41)]
            get(t, *b)
            out += b
        torch.cuda.synchronize()
        return out

    stream = torch.cuda.Stream()  # graph capture needs a non-default stream
    with torch.cuda.stream(stream):
        ref = []
        for i, n in zip(ids, sizes):
            hs = pr.pr_parareal_create(sde, sched, grid, 7, i, n)
            try:
                pr.pr_parareal_iterate(hs, 2)
                ref.append(states(lambda t, x, y, q: pr.pr_parareal_state(hs, t, x=x, y=y, q=q), n))
            finally:
                pr.pr_parareal_destroy(hs)
        for mode in (pr.PR_LAUNCH_BATCHED, pr.PR_LAUNCH_GRAPH):
            h = pr.pr_parareal_batch_create([sde] * 4, [sched] * 4, list(sizes), grid, 7, instances=list(ids))
            try:
                pr.pr_parareal_batch_iterate(h, 2, mode)
                for j, n in enumerate(sizes):
                    got = states(lambda t, x, y, q: pr.pr_parareal_batch_state(h, j, t, x=x, y=y, q=q), n)
                    assert all(torch.equal(a, b) for a, b in zip(got, ref[j])), (n, mode)
            finally:
                pr.pr_parareal_batch_destroy(h)


@pytest.mark.parametrize("longest", [64, 65])
def test_runs_of_equal_high_halves(longest):
    """Radix-sorted FP64 keys in runs that agree in their high halves, of 1, 2
    and the fix-up's longest run (64) and one key more (the complete sort), over
    tile edges and the ends, with repeated keys in them."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, rng = LONGEST + 4096 + 7, np.random.default_rng(5)
    lengths = np.resize([longest, 1, 2, 63, 64, 5], n)
    run = np.repeat(np.arange(n), lengths)[:n]
    x = 1.0 + run * 2.0 ** -20 + rng.integers(0, 40, n) * 2.0 ** -52
    x = x[rng.permutation(n)]
    print(f"runs of equal high halves up to {longest}", flush=True)
    d = torch.from_numpy(x).cuda()
    ws = torch.empty(pr.pr_restrict_workspace_size(n, 1, pr.PR_F64), dtype=torch.uint8, device="cuda")
    q = torch.zeros((1, 51), dtype=torch.float64, device="cuda")
    rank, perm = (torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(2))
    pr.pr_restrict_quantiles(d, pr.PR_F64, n, 1, 50, q, ws, rank=rank, perm=perm)
    torch.cuda.synchronize()
    p, r, v = OR.sort_ranks(x)
    assert np.array_equal(rank.cpu().numpy().view(np.uint32), r)
    assert np.array_equal(perm.cpu().numpy().view(np.uint32), p)
    assert np.array_equal(q[0].cpu().numpy(), OR.hazen_knots(v, 50))
