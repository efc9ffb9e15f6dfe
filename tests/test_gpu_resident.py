"""GPU: the resident sweep loop, which a split that fits the chip takes by
default, against per-sweep launches (JAC_OPT_GRID = 1 asks for them) and the
oracle.  Tiles, summation order and norms are the same, so every result is
bit-identical; the oracle bound is the per-sweep rounding of the row sums
(1e-12 relative per checked sweep, as for every other sweep path)."""
import threading

import numpy as np
import pytest
import scipy.sparse as sp

from gpu_util import B, get_x, make, need_gpu, rel_inf, set_x, sweep, torch
from oracle import ref
from paper_2112_02377_amd import workloads as W

pytestmark = pytest.mark.gpu


def banded(n, half, seed=3):
    """Rows reaching every column within `half`: 2 * half + 1 slots."""
    rng = np.random.default_rng(seed)
    off = [sp.diags(-rng.uniform(0.1, 1.0, n - d), d) for d in range(1, half + 1)]
    off = sp.csr_matrix(sum(off) + sum(o.T for o in off)) if off else sp.csr_matrix((n, n))
    A = (off + sp.diags(1.2 * np.asarray(abs(off).sum(axis=1)).ravel() + 0.1)).tocsr()
    A.sort_indices()
    return W.CSRSystem(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, rng.uniform(-1, 1, (1, n)))


def with_rhs(s, r):
    if r > 1:
        s.b = np.random.default_rng(9).uniform(-1, 1, (r, s.n))
    return s


# (system, split, parts, subdomains, right-hand sides): one tile, ragged last
# slices and tiles, each slot width (7, 14, 27), table and explicit columns
CASES = {
    "one-row": (lambda: banded(1, 0), 1, 1, None, 1),
    "one-tile": (lambda: banded(65, 1), 1, 1, None, 1),
    "tile-edge": (lambda: banded(512, 3), 1, 1, None, 1),
    "tile-edge-plus": (lambda: banded(513, 3), 1, 1, None, 2),
    "width-9": (lambda: banded(1500, 4), 1, 2, None, 1),
    "width-15": (lambda: banded(1100, 7), 2, 3, None, 1),
    "width-27": (lambda: banded(2000, 13), 1, 2, None, 4),
    "bands": (lambda: W.laplace7(13, workload=1), 1, 3, None, 1),
    "lists": (lambda: W.laplace7(17, workload=1), 2, 5, None, 2),
    "sub": (lambda: W.laplace7(16, workload=1), 3, 4, (2, 2, 2), 4),
    "fe-bands": (lambda: W.fe27(14, workload=3), 1, 3, None, 1),
    "fe-lists": (lambda: W.fe27(22, workload=3), 2, 4, None, 1),
    "fe-sub": (lambda: W.fe27(15, workload=3), 3, 4, (2, 2, 1), 2),
    "cube-sub": (lambda: W.fe_q1_cube(17), 3, 4, (2, 2, 2), 1),
}


def pair(name):
    build, mode, P, sub, r = CASES[name]
    s = with_rhs(build(), r)
    b = B()
    return s, r, [make(s, mode, P, sub, opts={b.JAC_OPT_GRID: g}) for g in (1, 0)]


@pytest.mark.parametrize("name", list(CASES))
def test_resident_loop_matches_per_sweep_launches(name):
    need_gpu()
    b = B()
    s, r, hs = pair(name)
    x0 = np.random.default_rng(5).uniform(-1, 1, (r, s.n))
    out = []
    for h in hs:
        set_x(h, x0)
        res = [sweep(h, 37, r), get_x(h, s.n, r)]
        if h is hs[1]:
            info = b.jac_get_info(h)
            assert info["loop_grid"] == info["ntiles"] + 4        # the resident loop ran: four deciding workgroups
        res.append(sweep(h, 7, r))                                # too short for it
        for norm in (b.JAC_NORM_L2_REL, b.JAC_NORM_INF_ABS):
            b.jac_set_x(h, None)
            st, sw, rr = b.jac_solve(h, 1e-9, 20000, norm)
            assert st == b.JAC_OK
            res += [sw, rr, get_x(h, s.n, r)]
        for maxit in (0, 8, 9, 20):                               # stops at the last residual
            b.jac_set_x(h, None)
            st, sw, rr = b.jac_solve(h, 0.0, maxit)
            res += [np.array(st), sw, rr, get_x(h, s.n, r)]
        b.jac_set_x(h, None)
        st, sw, rr = b.jac_solve(h, 1e-11, 4000, b.JAC_NORM_L2_REL, b.JAC_FP32_REFINE)
        res += [np.array(st), sw, rr, get_x(h, s.n, r)]
        out.append(res)
        b.jac_destroy(h)
    for k, (u, v) in enumerate(zip(*out)):
        assert np.array_equal(u, v), (name, k)
    for c in range(r):
        _, xr, hr = ref.sweeps(s.row_ptr, s.col_idx, s.vals, s.b[c], 37, x0=x0[c])
        assert rel_inf(out[1][1][c], xr) <= 1e-12
        assert np.all(np.abs(out[1][0][:, c] - hr) <= 1e-12 * np.maximum(hr, hr[0] * 1e-3))


def test_stop_at_once_and_divergence():
    need_gpu()
    b = B()
    s = W.laplace7(12, workload=1)
    bad = W.CSRSystem(s.row_ptr, s.col_idx, np.where(s.vals > 0, 0.5, s.vals), s.b, grid=s.grid)
    out = []
    for g in (1, 0):
        h = make(s, 1, 2, opts={b.JAC_OPT_GRID: g})
        b.jac_set_rhs(h, torch.zeros(s.n, dtype=torch.float64, device="cuda"))
        st, sw, rr = b.jac_solve(h, 1e-8, 1000)                   # b = 0, x = 0: x_0 passes
        assert (st, int(sw[0]), float(rr[0])) == (b.JAC_OK, 0, 0.0)
        b.jac_destroy(h)
        h = make(bad, 1, 2, opts={b.JAC_OPT_GRID: g})
        with pytest.raises(b.JacError) as e:
            b.jac_solve(h, 1e-8, 100000)
        assert e.value.status == b.JAC_E_DIVERGED
        out.append(get_x(h, s.n))
        b.jac_destroy(h)
    assert np.array_equal(out[0], out[1])


def test_many_launches_on_one_handle_after_a_new_split():
    # control words and ring are reused launch after launch, also when a new
    # split or precision lays them out differently
    need_gpu()
    b = B()
    s = W.laplace7(14, workload=1)
    h, hr = make(s, 1, 2), make(s, 1, 2, opts={b.JAC_OPT_GRID: 1})
    for k in range(12):
        mode, sub = ((1, None), (2, None), (3, (2, 2, 1)))[k % 3]
        got = []
        for hh in (h, hr):
            b.jac_partition(hh, mode, 4, sub)
            b.jac_set_x(hh, None)
            st, sw, rr = b.jac_solve(hh, 1e-6, 5000, b.JAC_NORM_L2_REL, b.JAC_FP32_REFINE if k % 2 else b.JAC_FP64)
            got.append((st, int(sw[0]), float(rr[0]), sweep(hh, 10 + k), get_x(hh, s.n)))
        assert got[0][:3] == got[1][:3]
        assert np.array_equal(got[0][3], got[1][3]) and np.array_equal(got[0][4], got[1][4])
    b.jac_destroy(h)
    b.jac_destroy(hr)


def test_the_loop_keeps_running_after_many_stops():
    # the workgroups that decide later sweeps must leave once an earlier sweep
    # stopped the last column, whatever they were waiting for: a launch that
    # runs out of patience sends its handle to per-sweep launches for good
    need_gpu()
    b = B()
    for s, prec in ((W.laplace7(10, workload=1), b.JAC_FP32_REFINE), (W.fe27(9, workload=3), b.JAC_FP64)):
        h = make(s, 1, 2)
        for k in range(150):
            b.jac_set_x(h, None)
            st, sw, rr = b.jac_solve(h, 10.0 ** -(3 + k % 7), 5000, b.JAC_NORM_L2_REL, prec)
            assert st == b.JAC_OK
        info = b.jac_get_info(h)
        assert info["loop_grid"] == info["ntiles"] + 4
        b.jac_destroy(h)


def test_threads_on_streams_of_their_own():
    need_gpu()
    b = B()
    s = W.laplace7(18, workload=1)
    h = make(s, 2, 3, opts={b.JAC_OPT_GRID: 1})
    b.jac_solve(h, 1e-8, 5000)
    want = get_x(h, s.n)
    b.jac_destroy(h)
    got, errors = [None] * 3, []

    def work(q):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                hh = make(s, 2, 3)
                for _ in range(3):
                    b.jac_set_x(hh, None)
                    b.jac_solve(hh, 1e-8, 5000)
                x = torch.empty(s.n, dtype=torch.float64, device="cuda")
                b.jac_get_x(hh, x)
                torch.cuda.current_stream().synchronize()
                got[q] = x.cpu().numpy()
                b.jac_destroy(hh)
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    ts = [threading.Thread(target=work, args=(q,)) for q in range(3)]
    [t.start() for t in ts]
    [t.join(60) for t in ts]
    assert not errors
    for g in got:
        assert np.array_equal(g, want[0])


@pytest.mark.parametrize("name,K,c", [("bands", 40, 7), ("lists", 9, 20), ("fe-bands", 33, 11), ("cube-sub", 25, 25)])
def test_adjoint_in_resident_launches(name, K, c):
    # forward, reverse sweeps and gradient against per-sweep launches (bit for
    # bit) and the oracle's full-storage reverse sweep (1e-10 relative to the
    # incoming gradient, the bar of every adjoint path)
    need_gpu()
    b = B()
    build, mode, P, sub, _ = CASES[name]
    s = build()
    g = np.random.default_rng(4).uniform(-1, 1, s.n)
    out = []
    for grid, mb in ((1, 4096), (0, 4096), (0, 4)):
        h = make(s, mode, P, sub, opts={b.JAC_OPT_GRID: grid, b.JAC_OPT_CKPT_MEM_MB: mb})
        gb = torch.empty(s.n, dtype=torch.float64, device="cuda")
        gv = torch.empty(s.nnz, dtype=torch.float64, device="cuda")
        b.jac_adjoint(h, K, c, torch.from_numpy(g).cuda(), gb, gv)
        out.append((gb.cpu().numpy(), gv.cpu().numpy(), get_x(h, s.n)[0]))
        b.jac_destroy(h)
    for k, o in enumerate(out[1:]):
        for u, v in zip(o, out[0]):
            assert np.array_equal(u, v), (name, k)
    _, gbo, gvo, xk = ref.adjoint(s.row_ptr, s.col_idx, s.vals, s.b[0], K, g)
    scale = np.abs(g).max()
    assert np.abs(out[1][0] - gbo).max() <= 1e-10 * scale and np.abs(out[1][1] - gvo).max() <= 1e-10 * scale
    assert rel_inf(out[1][2], xk) <= 1e-12


def mixed_widths(n, halves, seed=8):
    """Bands of changing width: row i reaches the columns within min(half_i, half_j)."""
    rng = np.random.default_rng(seed)
    half = np.repeat(halves, -(-n // len(halves)))[:n]
    rows, cols = [], []
    for i in range(n):
        j = np.arange(max(0, i - half[i]), min(n, i + half[i] + 1))
        j = j[np.abs(j - i) <= half[j]]
        rows.append(np.full(len(j), i))
        cols.append(j)
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    v = np.where(rows == cols, 30.0, rng.uniform(-1.0, -0.1, len(rows)))
    A = sp.csr_matrix((v, (rows, cols)), shape=(n, n))
    A.sort_indices()
    return W.CSRSystem(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, rng.uniform(-1, 1, (1, n)))


# slices as wide as the kernels' batches and narrower ones, in tables and in explicit columns; rows without some of
# their slice's table entries at the ends of the footprint
NONFINITE = {
    "widths-7": (lambda: mixed_widths(1500, (3, 1, 2)), 1, 2, None, 1),
    "widths-14": (lambda: mixed_widths(2100, (3, 6, 5)), 1, 2, None, 1),
    "widths-27": (lambda: mixed_widths(2600, (3, 10, 13, 6, 8)), 1, 3, None, 1),
    "widths-27-lists": (lambda: mixed_widths(2600, (3, 10, 13, 6, 8)), 2, 3, None, 2),
    "bands": CASES["bands"],
    "sub": CASES["sub"],
    "fe-bands": CASES["fe-bands"],
    "fe-lists": CASES["fe-lists"],
    "fe-sub": CASES["fe-sub"],
}


@pytest.mark.parametrize("name", list(NONFINITE))
def test_infinities_and_nans_spread_as_in_per_sweep_launches(name):
    # a zero times an infinity is not a zero: what a padded slot multiplies
    # decides which rows turn from infinite to NaN, and which stay finite
    need_gpu()
    b = B()
    build, mode, P, sub, r = NONFINITE[name]
    s = with_rhs(build(), r)
    n = s.n
    hs = [make(s, mode, P, sub, opts={b.JAC_OPT_GRID: g}) for g in (1, 0)]
    rng = np.random.default_rng(12)
    spots = [0, 1, 511, 512, n // 2, n - 64, n - 1] + list(rng.integers(0, n, 5))
    for q, at in enumerate(int(a) for a in spots):
        x0 = rng.uniform(-1, 1, (r, n))
        x0[q % r, at] = (np.inf, -np.inf, np.nan)[q % 3]
        out = []
        for h in hs:
            set_x(h, x0)
            out.append((sweep(h, 9, r), get_x(h, n, r)))
        info = b.jac_get_info(hs[1])
        assert info["loop_grid"] == info["ntiles"] + 4
        for u, v in zip(*out):
            assert np.array_equal(u, v, equal_nan=True), (name, at, x0[q % r, at])
        if r == 1:
            g = rng.uniform(-1, 1, n)
            g[at] = np.inf
            out = []
            for h in hs:
                b.jac_set_x(h, None)
                gb = torch.empty(n, dtype=torch.float64, device="cuda")
                gv = torch.empty(s.nnz, dtype=torch.float64, device="cuda")
                b.jac_adjoint(h, 10, 4, torch.from_numpy(g).cuda(), gb, gv)
                out.append((gb.cpu().numpy(), gv.cpu().numpy()))
            for u, v in zip(*out):
                assert np.array_equal(u, v, equal_nan=True), (name, at, "adjoint")
    for h in hs:
        b.jac_destroy(h)


@pytest.mark.parametrize("name", ["one-tile", "bands", "lists", "sub", "fe-bands", "fe-lists"])
def test_a_launch_that_gives_up_is_repeated_per_sweep(name):
    # no patience at all: the first value that is not there yet ends the
    # launch in every workgroup, and each call starts over per sweep; 32
    # loops later (64 after the next) the handle tries again
    need_gpu()
    b = B()
    s, r, hs = pair(name)
    h = hs[1]
    x0 = np.random.default_rng(5).uniform(-1, 1, (r, s.n))
    g = torch.from_numpy(np.random.default_rng(4).uniform(-1, 1, s.n)).cuda()
    gb = torch.empty(s.n, dtype=torch.float64, device="cuda")
    gv = torch.empty(s.nnz, dtype=torch.float64, device="cuda")

    def fixed(h):
        set_x(h, x0)
        return [sweep(h, 37, r), get_x(h, s.n, r)]

    def solve(h, prec=b.JAC_FP64, tol=1e-9):
        b.jac_set_x(h, None)
        st, sw, rr = b.jac_solve(h, tol, 20000, b.JAC_NORM_L2_REL, prec)
        return [np.array(st), sw, rr, get_x(h, s.n, r)]

    def refine(h):
        return solve(h, b.JAC_FP32_REFINE, 1e-11)

    def adjoint(h):
        b.jac_adjoint(h, 30, 7, g, gb, gv)
        return [gb.cpu().numpy(), gv.cpu().numpy(), get_x(h, s.n, r)]

    for call in (fixed, solve, refine) + ((adjoint,) if r == 1 else ()):
        want = call(hs[0])
        ran = b.jac_get_info(h)["resident_loops"]
        got = call(h)
        assert b.jac_get_info(h)["resident_loops"] > ran, call.__name__        # the loop takes this call
        ran = b.jac_get_info(h)["resident_loops"]
        b.jac_set_option(h, b.JAC_OPT_LOOP_WAIT, 0)
        gave_up = call(h)
        b.jac_set_option(h, b.JAC_OPT_LOOP_WAIT, 2000000)
        assert b.jac_get_info(h)["resident_loops"] == ran, call.__name__
        for k, (u, v, w) in enumerate(zip(want, got, gave_up)):
            assert np.array_equal(u, v) and np.array_equal(u, w), (name, call.__name__, k)
        n = 0
        while b.jac_get_info(h)["resident_loops"] == ran:                      # per sweep until it tries again
            assert n < 80
            b.jac_sweep(h, 8, None)
            n += 1
        got = call(h)
        for k, (u, v) in enumerate(zip(want, got)):
            assert np.array_equal(u, v), (name, call.__name__, k)
    assert b.jac_get_info(hs[0])["resident_loops"] == 0
    for h in hs:
        b.jac_destroy(h)


TICKS = []


def busy_stream(ms):
    """Puts about `ms` of device work on the current stream and returns an event behind it."""
    if not TICKS:                                                 # of the clock that _sleep counts, per ms
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for k in range(2):
            e[0].record()
            torch.cuda._sleep(2000000)
            e[1].record()
            torch.cuda.synchronize()
        TICKS.append(2000000 / e[0].elapsed_time(e[1]))
    torch.cuda._sleep(int(ms * TICKS[0]))
    e = torch.cuda.Event()
    e.record()
    return e


def test_fixed_sweeps_do_not_wait_for_the_device():
    # jac_sweep and jac_sweep_checkpointed return with their work on the stream, also in a resident launch
    need_gpu()
    b = B()
    s = W.laplace7(20, workload=1)
    h = make(s, 1, 2)
    hist = torch.zeros(50, dtype=torch.float64, device="cuda")
    x = torch.empty(s.n, dtype=torch.float64, device="cuda")
    b.jac_sweep(h, 50, hist)                                      # first calls allocate, which waits
    b.jac_sweep_checkpointed(h, 50, 10)
    torch.cuda.synchronize()
    b.jac_set_x(h, None)
    before = busy_stream(500)
    b.jac_sweep(h, 50, hist)
    b.jac_get_x(h, x)
    assert not before.query()
    torch.cuda.synchronize()
    b.jac_set_x(h, None)
    before = busy_stream(500)
    b.jac_sweep_checkpointed(h, 50, 10)
    assert not before.query()
    torch.cuda.synchronize()
    assert b.jac_get_info(h)["resident_loops"] == 4
    _, xr, hr = ref.sweeps(s.row_ptr, s.col_idx, s.vals, s.b[0], 50)
    assert rel_inf(x.cpu().numpy(), xr) <= 1e-12 and rel_inf(get_x(h, s.n)[0], xr) <= 1e-12
    assert np.all(np.abs(hist.cpu().numpy() - hr) <= 1e-12 * np.maximum(hr, hr[0] * 1e-3))
    b.jac_destroy(h)


@pytest.mark.parametrize("name", list(CASES))
def test_fixed_sweeps_of_launches_that_give_up_are_done_again_on_the_device(name):
    # several on the stream before the host can know, infinities among x
    need_gpu()
    b = B()
    s, r, hs = pair(name)
    x0 = np.random.default_rng(5).uniform(-1, 1, (r, s.n))
    x0[0, s.n // 2] = np.inf
    b.jac_set_option(hs[1], b.JAC_OPT_LOOP_WAIT, 0)
    out = []
    for h in hs:
        set_x(h, x0)
        hist = [torch.zeros(K * r, dtype=torch.float64, device="cuda") for K in (8, 21)]
        for hi in hist:
            b.jac_sweep(h, hi.numel() // r, hi)
        x = torch.empty(s.n * r, dtype=torch.float64, device="cuda")
        b.jac_get_x(h, x)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in hist + [x]])
    assert b.jac_get_info(hs[1])["resident_loops"] == 0
    for k, (u, v) in enumerate(zip(*out)):
        assert np.array_equal(u, v, equal_nan=True), (name, k)
    for h in hs:
        b.jac_destroy(h)


def test_loops_longer_than_one_launch():
    # a resident launch holds at most 65536 sweeps: longer loops go on in the
    # next one, from the same iterate, with the stopped columns left alone
    need_gpu()
    b = B()
    n = 200
    A = sp.diags([2.0 * np.ones(n), -np.ones(n - 1), -np.ones(n - 1)], [0, 1, -1]).tocsr()
    A.sort_indices()
    rng = np.random.default_rng(2)
    rhs = np.stack([np.sin(np.pi * np.arange(1, n + 1) / (n + 1)),            # some 150000 sweeps
                    np.sin(70 * np.pi * np.arange(1, n + 1) / (n + 1))])      # some 30
    s = W.CSRSystem(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, rhs)
    s1 = W.CSRSystem(s.row_ptr, s.col_idx, s.vals, rng.uniform(-1, 1, (1, n)))
    hs = [make(s, 1, 1, opts={b.JAC_OPT_GRID: g}) for g in (1, 0)]
    h1 = [make(s1, 1, 1, opts={b.JAC_OPT_GRID: g}) for g in (1, 0)]
    out = []
    for h, g in zip(hs, h1):
        res = [sweep(h, 70000, 2), get_x(h, n, 2)]
        for tol, maxit in ((1e-8, 1000000), (1e-8, 140000), (1e-2, 66000), (1e-8, 65536), (1e-8, 65537)):
            b.jac_set_x(h, None)
            st, sw, rr = b.jac_solve(h, tol, maxit)
            res += [np.array(st), sw, rr, get_x(h, n, 2)]
        assert res[2] == b.JAC_OK and 131072 < res[3][0] < 200000 and res[3][1] < 100 and res[6] == b.JAC_NOT_CONVERGED
        b.jac_set_option(g, b.JAC_OPT_INNER_TOL, 1)
        b.jac_set_option(g, b.JAC_OPT_INNER_MAX, 80000)
        st, sw, rr = b.jac_solve(g, 1e-3, 200000, b.JAC_NORM_L2_REL, b.JAC_FP32_REFINE)
        assert int(sw[0]) >= 80000
        res += [np.array(st), sw, rr, get_x(g, n)]
        gb = torch.empty(n, dtype=torch.float64, device="cuda")
        gv = torch.empty(s1.nnz, dtype=torch.float64, device="cuda")
        b.jac_adjoint(g, 70000, 5000, torch.from_numpy(rhs[1]).cuda(), gb, gv)
        res += [gb.cpu().numpy(), gv.cpu().numpy(), get_x(g, n)]
        out.append(res)
    # 2 launches of sweeps; 3, 3, 1 or 2, 1 and 2 of solves at least; the same of the refinement and the forward
    assert b.jac_get_info(hs[1])["resident_loops"] >= 11 and b.jac_get_info(h1[1])["resident_loops"] >= 4
    for k, (u, v) in enumerate(zip(*out)):
        assert np.array_equal(u, v), k
    for h in hs + h1:
        b.jac_destroy(h)


@pytest.mark.parametrize("edge,joins", [(16, True), (64, False)])
def test_a_loop_does_not_wait_for_other_streams(edge, joins):
    # a resident launch that its stream holds back must not hold back the
    # loops of other streams: they are on the device beside it where both fit
    # whole, else launched per sweep until it has ended
    need_gpu()
    b = B()
    s = W.laplace7(edge, workload=1)
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    hs = []
    for st in (one, two):
        with torch.cuda.stream(st):
            hs.append(make(s, 1, 2))
            b.jac_sweep(hs[-1], 50, None)
        torch.cuda.synchronize()
    with torch.cuda.stream(two):
        b.jac_set_x(hs[1], None)
        st, sw, rr = b.jac_solve(hs[1], 1e-3, 5000)
        want = get_x(hs[1], s.n)
    torch.cuda.synchronize()

    def ran():
        return [b.jac_get_info(h)["resident_loops"] for h in hs]

    assert ran() == [1, 2]
    with torch.cuda.stream(one):
        before = busy_stream(500)
        b.jac_sweep(hs[0], 50, None)
        b.jac_sweep(hs[0], 50, None)
    with torch.cuda.stream(two):
        b.jac_set_x(hs[1], None)
        got = b.jac_solve(hs[1], 1e-3, 5000)
    assert not before.query()
    assert got == (st, sw, rr) and np.array_equal(get_x(hs[1], s.n), want)
    torch.cuda.synchronize()
    assert ran() == [3, 3 if joins else 2]
    with torch.cuda.stream(two):
        b.jac_solve(hs[1], 1e-4, 5000)
        assert ran() == [3, 4 if joins else 3]
        b.jac_destroy(hs.pop(0))
        b.jac_sweep(hs[0], 50, None)
    torch.cuda.synchronize()
    assert ran() == [5 if joins else 4]
    b.jac_destroy(hs[0])


def test_autotune_keeps_the_resident_loop(tmp_path, monkeypatch):
    # a tuned handle of a system that fits the device stays on the loop it
    # runs by default, from the cache too, and with a cache of a time when
    # the loop was not among the candidates; a grid of the caller's own keeps
    # per-sweep launches
    need_gpu()
    b = B()
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("JAC_TUNE_CACHE", str(cache))
    s = W.laplace7(24, workload=1)

    def tuned(grid=0):
        h = make(s, 2, 4, opts={b.JAC_OPT_GRID: grid})
        b.jac_autotune(h, 20)
        ran = b.jac_get_info(h)["resident_loops"]
        b.jac_set_x(h, None)
        st, sw, rr = b.jac_solve(h, 1e-8, 10000)
        info = b.jac_get_info(h)
        x = get_x(h, s.n)
        return h, info["resident_loops"] - ran, int(sw[0]), x, len(cache.read_text().splitlines())

    _, xr, kr, _ = ref.solve(s.row_ptr, s.col_idx, s.vals, s.b[0], 1e-8, 10000)
    handles = []
    for k, (grid, loops, lines) in enumerate(((0, 1, 3), (0, 1, 3), (1, 0, 3), (0, 1, 3), (0, 1, 6))):
        if k == 4:
            cache.write_text(cache.read_text().replace("|1 1 ", "|1 0 ").replace("|2 1 ", "|2 0 "))
        h, ran, sweeps, x, stored = tuned(grid)
        handles.append(h)
        assert (ran, sweeps, stored) == (loops, kr, lines), k
        assert rel_inf(x[0], xr) <= 1e-10
        if grid == 0:
            assert b.jac_get_option(h, b.JAC_OPT_BLOCK) == 256 and b.jac_get_option(h, b.JAC_OPT_GRID) in (1, 2)
    b.jac_set_option(handles[0], b.JAC_OPT_GRID, 1)
    ran = b.jac_get_info(handles[0])["resident_loops"]
    b.jac_set_x(handles[0], None)
    b.jac_solve(handles[0], 1e-8, 10000)
    assert b.jac_get_info(handles[0])["resident_loops"] == ran
    for h in handles:
        b.jac_destroy(h)


@pytest.mark.parametrize("grid", [0, 1])
def test_adjoint_allocates_what_its_route_needs(grid):
    # per sweep: all iterates, the mu of a segment; resident: all iterates, all mu, the ring of eight
    need_gpu()
    b = B()
    s = W.diffusion_adjoint(48)
    K, c = 120, 40
    g = torch.from_numpy(np.random.default_rng(4).uniform(-1, 1, s.n)).cuda()
    gb, gv = torch.empty(s.n, dtype=torch.float64, device="cuda"), torch.empty(s.nnz, dtype=torch.float64, device="cuda")
    h = make(s, 1, 1, opts={b.JAC_OPT_GRID: grid})
    vec = 8 * s.n
    b.jac_adjoint(h, 0, 1, g, gb, gv)                              # the transposed layout and the small buffers
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    b.jac_adjoint(h, K, c, g, gb, gv)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    need = (K + 1 + (K + 8 if grid == 0 else c + 2)) * vec
    assert used <= need + 24 * vec, (used / vec, need / vec)       # allocations are rounded up
    assert b.jac_get_info(h)["resident_loops"] == (2 if grid == 0 else 0)
    b.jac_destroy(h)


@pytest.mark.parametrize("r", [1, 2, 4])
@pytest.mark.parametrize("half", [2, 4, 6, 9, 13])
@pytest.mark.parametrize("tables", [0, 1])
def test_every_kernel_of_the_loop(half, r, tables):
    # 5, 9, 13, 19 and 27 slots, from a shift table and as explicit columns,
    # FP64 and FP32: each runs, and gives the bits of per-sweep launches
    need_gpu()
    b = B()
    s = with_rhs(banded(1700, half), r)
    x0 = np.random.default_rng(5).uniform(-1, 1, (r, s.n))
    out = []
    for g in (1, 0):
        h = make(s, 2, 3, opts={b.JAC_OPT_GRID: g, b.JAC_OPT_SHIFT_TABLES: tables})
        b.jac_partition(h, 2, 3, None)
        assert b.jac_get_info(h)["col_format"] == (4 if tables else 2)
        set_x(h, x0)
        res = [sweep(h, 20, r), get_x(h, s.n, r)]
        for prec in (b.JAC_FP64, b.JAC_FP32_REFINE):
            b.jac_set_x(h, None)
            st, sw, rr = b.jac_solve(h, 1e-10, 5000, b.JAC_NORM_L2_REL, prec)
            assert st == b.JAC_OK
            res += [sw, rr, get_x(h, s.n, r)]
        ran = b.jac_get_info(h)["resident_loops"]
        assert ran == 0 if g else ran >= 3, ran
        out.append(res)
        b.jac_destroy(h)
    for k, (u, v) in enumerate(zip(*out)):
        assert np.array_equal(u, v), k


@pytest.mark.parametrize("half", [3, 4, 6, 9, 13])
def test_every_reverse_kernel_of_the_loop(half):
    need_gpu()
    b = B()
    s = banded(1700, half)
    g = np.random.default_rng(4).uniform(-1, 1, s.n)
    out = []
    for grid in (1, 0):
        h = make(s, 1, 3, opts={b.JAC_OPT_GRID: grid})
        gb = torch.empty(s.n, dtype=torch.float64, device="cuda")
        gv = torch.empty(s.nnz, dtype=torch.float64, device="cuda")
        b.jac_adjoint(h, 25, 6, torch.from_numpy(g).cuda(), gb, gv)
        assert b.jac_get_info(h)["resident_loops"] == (0 if grid else 2)       # forward and reverse
        out.append((gb.cpu().numpy(), gv.cpu().numpy(), get_x(h, s.n)))
        b.jac_destroy(h)
    for k, (u, v) in enumerate(zip(*out)):
        assert np.array_equal(u, v), k


def test_loops_of_threads_are_resident():
    need_gpu()
    b = B()
    s = W.laplace7(18, workload=1)
    ran, errors = [0] * 4, []

    def work(q):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                h = make(s, 2, 3)
                for _ in range(5):
                    b.jac_set_x(h, None)
                    b.jac_solve(h, 1e-8, 5000)
                ran[q] = b.jac_get_info(h)["resident_loops"]
                b.jac_destroy(h)
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    ts = [threading.Thread(target=work, args=(q,)) for q in range(4)]
    [t.start() for t in ts]
    [t.join(60) for t in ts]
    assert not errors and ran == [5] * 4


@pytest.mark.parametrize("edge,r,least", [(48, 1, 8), (64, 1, 8), (72, 1, 16), (80, 1, 16), (64, 4, 16), (48, 4, 8)])
def test_short_loops_of_large_systems_are_launched_per_sweep(edge, r, least):
    # where filling the ring and loading the matrix take longer than the sweeps gain
    need_gpu()
    b = B()
    s = with_rhs(W.laplace7(edge, workload=1), r)
    out = []
    for g in (1, 0):
        h = make(s, 1, 4, opts={b.JAC_OPT_GRID: g})
        res = []
        for k, loops in ((least - 1, 0), (least, 1 - g)):
            ran = b.jac_get_info(h)["resident_loops"]
            res += [sweep(h, k, r)]
            assert b.jac_get_info(h)["resident_loops"] == ran + loops
        out.append(res + [get_x(h, s.n, r)])
        b.jac_destroy(h)
    for u, v in zip(*out):
        assert np.array_equal(u, v)


def test_sweeps_are_not_captured():
    # a resident launch carries numbers that must not come again, so a graph
    # of it would be wrong from its second replay on: a capture is refused,
    # as it is by the per-sweep loop, and the handle goes on
    import ctypes
    need_gpu()
    b = B()
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
    hip = ctypes.CDLL(path)
    s = W.laplace7(16, workload=1)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        h = make(s, 1, 2)
        b.jac_sweep(h, 20, None)
        st.synchronize()
        want = get_x(h, s.n)
        graph = ctypes.c_void_p()
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(st.cuda_stream), 2) == 0      # relaxed
        with pytest.raises(b.JacError) as e:
            b.jac_sweep(h, 20, None)
        assert hip.hipStreamEndCapture(ctypes.c_void_p(st.cuda_stream), ctypes.byref(graph)) == 0
        assert e.value.status == b.JAC_E_HIP and hip.hipGraphDestroy(graph) == 0
        torch.cuda.synchronize()
        assert np.array_equal(get_x(h, s.n), want)
        b.jac_set_x(h, None)
        b.jac_sweep(h, 20, None)
        assert np.array_equal(get_x(h, s.n), want)
        b.jac_destroy(h)


def test_no_thread_is_kept_out_by_the_loops_of_another():
    # two threads, one solve after the other, of which only one fits the
    # device: each gets its turns (a call is two solves long then; without a
    # queue the longest took more than ten)
    need_gpu()
    import time
    b = B()
    s = W.laplace7(64, workload=1)
    took, errors = [[], []], []
    start = threading.Barrier(2)

    def work(q):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                h = make(s, 1, 4)
                b.jac_solve(h, 1e-3, 100000)
                start.wait(30)
                end = time.perf_counter() + 1.5
                while time.perf_counter() < end:
                    t = time.perf_counter()
                    b.jac_set_x(h, None)
                    b.jac_solve(h, 1e-3, 100000)
                    took[q].append(time.perf_counter() - t)
                b.jac_destroy(h)
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    ts = [threading.Thread(target=work, args=(q,)) for q in range(2)]
    [t.start() for t in ts]
    [t.join(60) for t in ts]
    assert not errors
    alone = min(took[0] + took[1])
    for t in took:
        assert np.percentile(t, 98) < 8 * alone and sum(t) < 3.0, (alone, np.percentile(t, 98), max(t))
