"""GPU: the checkpointed adjoint (jac_adjoint) and the autograd Function,
against the oracle's full-storage reverse sweep, the dot-product identity and
central finite differences."""
import numpy as np
import pytest

from gpu_util import B, get_x, make, need_gpu, rel_inf, torch
from oracle import ref
from paper_2112_02377_amd import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def run_adjoint(h, K, c, g, n, nnz):
    b = B()
    gb = torch.empty(n, dtype=torch.float64, device="cuda")
    gv = torch.empty(nnz, dtype=torch.float64, device="cuda")
    b.jac_adjoint(h, K, c, dev(g), gb, gv)
    torch.cuda.synchronize()
    return gb.cpu().numpy(), gv.cpu().numpy()


@pytest.mark.parametrize("mode,P,sub,K,c", [(1, 1, None, 60, 7), (1, 3, None, 45, 45), (2, 4, None, 33, 10),
                                            (3, 4, (2, 2, 1), 50, 8), (1, 2, None, 1, 5)])
def test_adjoint_matches_full_storage_oracle(mode, P, sub, K, c):
    need_gpu()
    b = B()
    s = W.diffusion_adjoint(10)
    t = s.extra["x_target"]
    h = make(s, mode, P, sub)
    st, xo, _ = ref.sweeps(s.row_ptr, s.col_idx, s.vals, s.b[0], K)
    g = xo - t
    gb, gv = run_adjoint(h, K, c, g, s.n, s.nnz)
    sto, gbo, gvo, xk = ref.adjoint(s.row_ptr, s.col_idx, s.vals, s.b[0], K, g)
    assert np.abs(gb - gbo).max() <= 1e-10 * np.abs(gbo).max()
    assert np.abs(gv - gvo).max() <= 1e-10 * np.abs(gvo).max()
    # the handle keeps x_K
    assert rel_inf(get_x(h, s.n)[0], xk) <= 1e-12
    b.jac_destroy(h)


@pytest.mark.parametrize("tile", [64, 448, 8192])
def test_gradient_pass_over_tile_sizes(tile):
    # tiles of one slice, of no multiple of a workgroup's four and of more
    # slices than the launch has waves for; 7- and 27-entry rows (one batch
    # and four), a last segment of its own length
    need_gpu()
    b = B()
    for s in (W.diffusion_adjoint(23), W.fe27(15)):
        K = 17
        g = np.random.default_rng(6).uniform(-1, 1, s.n)
        h = make(s, 1, 1, opts={b.JAC_OPT_TILE_ROWS: tile})
        gb, gv = run_adjoint(h, K, 5, g, s.n, s.nnz)
        _, gbo, gvo, _ = ref.adjoint(s.row_ptr, s.col_idx, s.vals, s.b[0], K, g)
        assert np.abs(gb - gbo).max() <= 1e-10 * np.abs(gbo).max(), tile
        assert np.abs(gv - gvo).max() <= 1e-10 * np.abs(gvo).max(), tile
        b.jac_destroy(h)


def test_adjoint_of_nonsymmetric_paper_example():
    need_gpu()
    from test_oracle_pins import fig_csr
    b = B()
    IA, JA, AA, dense = fig_csr()
    rng = np.random.default_rng(21)
    rhs = rng.uniform(-1, 1, 5)
    g = rng.uniform(-1, 1, 5)
    h = b.jac_create(5, IA, JA, AA, 1, rhs)
    for K, c in ((9, 4), (12, 12), (7, 1)):
        gb, gv = run_adjoint(h, K, c, g, 5, len(AA))
        sto, gbo, gvo, _ = ref.adjoint(IA, JA, AA, rhs, K, g)
        assert np.abs(gb - gbo).max() <= 1e-12 * np.abs(gbo).max()
        assert np.abs(gv - gvo).max() <= 1e-12 * np.abs(gvo).max()
    b.jac_destroy(h)


def test_dot_product_identity_on_device():
    # <S_K v, w> = <v, S_K^T w>, both sides computed by the library
    need_gpu()
    b = B()
    s = W.diffusion_adjoint(12)
    rng = np.random.default_rng(8)
    v = rng.uniform(-1, 1, s.n)
    w = rng.uniform(-1, 1, s.n)
    K = 80
    h = make(s, 2, 3)
    b.jac_set_rhs(h, dev(v))
    b.jac_set_x(h, None)
    b.jac_sweep(h, K)
    Sv = get_x(h, s.n)[0]
    STw, _ = run_adjoint(h, K, 16, w, s.n, s.nnz)
    lhs, rhs = Sv @ w, v @ STw
    assert abs(lhs - rhs) <= 1e-12 * max(abs(lhs), 1.0)
    b.jac_destroy(h)


def test_autograd_theta_gradient_matches_oracle_chain_rule():
    need_gpu()
    from paper_2112_02377_amd.autograd import JacobiK, diffusion_values
    s = W.diffusion_adjoint(8)
    t = dev(s.extra["x_target"])
    K, c = 70, 9
    h = make(s, 1, 2)
    theta = dev(s.extra["theta"]).requires_grad_(True)
    vals = diffusion_values(theta, s.grid, s.row_ptr, s.extra["slot"])
    assert np.array_equal(vals.detach().cpu().numpy(), s.vals)     # same assembly as the generator
    x = JacobiK.apply(vals, dev(s.b[0]), h, K, c)
    loss = 0.5 * ((x - t) ** 2).sum()
    loss.backward()
    gth = theta.grad.cpu().numpy()
    st, xo, _ = ref.sweeps(s.row_ptr, s.col_idx, s.vals, s.b[0], K)
    _, gbo, gvo, _ = ref.adjoint(s.row_ptr, s.col_idx, s.vals, s.b[0], K, xo - s.extra["x_target"])
    gth_o = ref.theta_grad(s.extra["theta"], s.grid, s.row_ptr, s.extra["slot"], gvo)
    assert np.abs(gth - gth_o).max() <= 1e-10 * np.abs(gth_o).max()
    B().jac_destroy(h)


def test_full_size_theta_gradient_against_central_differences():
    """64^3 conductivities, K = 400 sweeps, checkpoint every 20: dL/dtheta from
    the autograd Function at 32 seeded entries against central differences
    (step 1e-6) of the same forward."""
    need_gpu()
    from paper_2112_02377_amd.autograd import JacobiK, diffusion_values
    b = B()
    s = W.diffusion_adjoint(64)
    K, c, hstep = 400, 20, 1e-6
    tnp = s.extra["x_target"]
    t = dev(tnp)
    h = make(s, 1, 1)
    theta = dev(s.extra["theta"]).requires_grad_(True)
    vals = diffusion_values(theta, s.grid, s.row_ptr, s.extra["slot"])
    x = JacobiK.apply(vals, dev(s.b[0]), h, K, c)
    (0.5 * ((x - t) ** 2).sum()).backward()
    g = theta.grad.cpu().numpy()
    fd = []
    for m in s.extra["probes"]:
        xs = []
        for sign in (1, -1):
            th = s.extra["theta"].copy()
            th[m] += sign * hstep
            v = W.diffusion_values(th, 64, 64, 64, s.row_ptr, s.extra["slot"])
            b.jac_set_values(h, dev(v))
            b.jac_set_x(h, None)
            b.jac_sweep(h, K)
            xs.append(get_x(h, s.n)[0])
        fd.append(np.sum((xs[0] - xs[1]) * (xs[0] + xs[1] - 2 * tnp)) / (4 * hstep))
    fd = np.array(fd)
    gp = g[s.extra["probes"]]
    assert np.all(np.abs(gp - fd) <= 1e-5 * np.maximum(np.abs(fd), 1e-3 * np.abs(fd).max())), (gp, fd)
    b.jac_destroy(h)


def test_checkpointed_forward_is_reused_and_invalidated():
    need_gpu()
    b = B()
    s = W.diffusion_adjoint(12)
    K, c = 90, 7
    h = make(s, 2, 3)
    st, xo, _ = ref.sweeps(s.row_ptr, s.col_idx, s.vals, s.b[0], K)
    g = xo - s.extra["x_target"]
    # forward kept on the device: the same iterate as K plain sweeps
    b.jac_sweep_checkpointed(h, K, c)
    assert rel_inf(get_x(h, s.n)[0], xo) <= 1e-12
    gen = b.jac_get_info(h)["state_gen"]
    gb1, gv1 = run_adjoint(h, K, c, g, s.n, s.nnz)          # reuses the checkpoints
    assert b.jac_get_info(h)["state_gen"] == gen
    b.jac_set_x(h, None)                                    # any change invalidates them
    assert b.jac_get_info(h)["state_gen"] > gen
    gb2, gv2 = run_adjoint(h, K, c, g, s.n, s.nnz)          # takes them again
    assert np.array_equal(gb1, gb2) and np.array_equal(gv1, gv2)
    sto, gbo, gvo, _ = ref.adjoint(s.row_ptr, s.col_idx, s.vals, s.b[0], K, g)
    assert np.abs(gb1 - gbo).max() <= 1e-10 * np.abs(gbo).max()
    assert np.abs(gv1 - gvo).max() <= 1e-10 * np.abs(gvo).max()
    # a different K or stride does not reuse them; new values are picked up
    b.jac_sweep_checkpointed(h, K, c)
    gb3, _ = run_adjoint(h, K - 5, c, g, s.n, s.nnz)
    _, gbo3, _, _ = ref.adjoint(s.row_ptr, s.col_idx, s.vals, s.b[0], K - 5, g)
    assert np.abs(gb3 - gbo3).max() <= 1e-10 * np.abs(gbo3).max()
    b.jac_sweep_checkpointed(h, K, c)
    v2 = s.vals * 1.01
    b.jac_set_values(h, dev(v2))
    gb4, gv4 = run_adjoint(h, K, c, g, s.n, s.nnz)
    _, gbo4, gvo4, _ = ref.adjoint(s.row_ptr, s.col_idx, v2, s.b[0], K, g)
    assert np.abs(gv4 - gvo4).max() <= 1e-10 * np.abs(gvo4).max()
    b.jac_destroy(h)


def test_autograd_backward_after_the_handle_was_used_again():
    # backward restores the system when the handle was used in between
    need_gpu()
    from paper_2112_02377_amd.autograd import JacobiK, diffusion_values
    b = B()
    s = W.diffusion_adjoint(8)
    t = dev(s.extra["x_target"])
    h = make(s, 1, 2)
    grads = []
    for touch in (False, True):
        theta = dev(s.extra["theta"]).requires_grad_(True)
        vals = diffusion_values(theta, s.grid, s.row_ptr, s.extra["slot"])
        x = JacobiK.apply(vals, dev(s.b[0]), h, 60, 9)
        if touch:
            b.jac_set_values(h, dev(s.vals * 2.0))
            b.jac_set_x(h, None)
            b.jac_sweep(h, 5)
        (0.5 * ((x - t) ** 2).sum()).backward()
        grads.append(theta.grad.cpu().numpy())
    assert np.array_equal(grads[0], grads[1])
    b.jac_destroy(h)


def test_stored_and_recomputed_iterates_give_identical_gradients():
    # all K + 1 iterates fit the default cap: stored, nothing recomputed; a
    # 1 MiB cap forces checkpoints every c sweeps and recomputed segments
    need_gpu()
    b = B()
    s = W.diffusion_adjoint(10)
    K, c = 300, 16
    st, xo, _ = ref.sweeps(s.row_ptr, s.col_idx, s.vals, s.b[0], K)
    g = xo - s.extra["x_target"]
    out = []
    for cap in (4096, 1):
        h = make(s, 2, 3, opts={b.JAC_OPT_CKPT_MEM_MB: cap})
        gb, gv = run_adjoint(h, K, c, g, s.n, s.nnz)
        out.append((gb, gv, get_x(h, s.n)[0]))
        b.jac_destroy(h)
    assert all(np.array_equal(u, v) for u, v in zip(out[0], out[1]))
    sto, gbo, gvo, xk = ref.adjoint(s.row_ptr, s.col_idx, s.vals, s.b[0], K, g)
    assert np.abs(out[0][0] - gbo).max() <= 1e-10 * np.abs(gbo).max()
    assert np.abs(out[0][1] - gvo).max() <= 1e-10 * np.abs(gvo).max()
    assert rel_inf(out[0][2], xk) <= 1e-12
    # a cap too small for either layout is refused
    h = make(s, 1, 1, opts={b.JAC_OPT_CKPT_MEM_MB: 1})
    with pytest.raises(b.JacError) as e:
        b.jac_adjoint(h, 3000, 3000, dev(g), torch.empty(s.n, dtype=torch.float64, device="cuda"),
                      torch.empty(s.nnz, dtype=torch.float64, device="cuda"))
    assert e.value.status == b.JAC_E_INVALID
    b.jac_destroy(h)


def test_full_size_stored_and_recomputed_agree():
    # 64^3, K = 400, segments of 20: 841 MB of iterates under the default cap
    # against checkpoints every 20 sweeps under a 200 MiB cap
    need_gpu()
    b = B()
    s = W.diffusion_adjoint(64)
    g = np.random.default_rng(9).uniform(-1, 1, s.n)
    res = []
    for cap in (4096, 200):
        h = make(s, 1, 1, opts={b.JAC_OPT_CKPT_MEM_MB: cap})
        b.jac_sweep_checkpointed(h, 400, 20)
        res.append(run_adjoint(h, 400, 20, g, s.n, s.nnz))
        b.jac_destroy(h)
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])
