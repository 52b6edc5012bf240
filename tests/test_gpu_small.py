"""The projected problems of the restarts at the edges of their launch shapes: one or several rows
per lane (64, 128, 192), matrices that just fit in LDS or do not, odd and even orders."""
import numpy as np
import pytest

from lattice_inputs import gaussian_spinor
from oracle import dirac

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,m,k", [
    ("g5m", 9, 1), ("g5m", 63, 20), ("g5m", 64, 21), ("g5m", 127, 20), ("g5m", 128, 64), ("g5m", 139, 30),
    ("g5m", 140, 30), ("g5m", 192, 40), ("g5m", 210, 199), ("mdagm", 20, 1), ("mdagm", 33, 16), ("mdagm", 64, 20),
    ("mdagm", 141, 20), ("mdagm", 142, 20), ("mdagm", 143, 40), ("mdagm", 202, 141)])
def test_first_solve_over_basis_sizes(gpu_ctx, c1_config, kind, m, k):
    """A restarted first solve converges (FP64 residual by the oracle's matrix), and the kept
    vectors are orthonormal with the residual norms that the handle reports.  The kappa is off
    critical, so that small bases converge too.  Residual norms of unit vectors are compared to
    1e-11, the rounding of the Rayleigh quotient (1e-15 ||A||) over the smallest norm kept apart."""
    from paper_0901_3163_amd import deflan
    dims, U, kappa = c1_config["dims"], c1_config["links"], 0.13
    ora = dirac.WilsonOperator(U, dims, kappa)
    op = deflan.Operator(gpu_ctx, dims, U, kappa, deflan.DL_G5M if kind == "g5m" else deflan.DL_MDAGM)
    b = gaussian_spinor(dims, 300 + m)
    x, eig, st = op.solve_first(b, m, k, 1e-10, max_mvp=20000)
    assert st["status"] == 0, st
    r = b.ravel() - ora.M(x.ravel())
    assert np.linalg.norm(r) <= 1.0001e-10 * np.linalg.norm(b)
    ev, res = eig.info()
    Y = eig.vectors().reshape(k, -1)
    gram = Y.conj() @ Y.T
    assert np.max(np.abs(gram - np.eye(k))) < 1e-10
    for i in sorted({0, k // 2, k - 1}):
        a = ora.g5M(Y[i]) if kind == "g5m" else ora.Mdag(ora.M(Y[i]))
        assert abs(np.vdot(Y[i], a).real - ev[i]) < 1e-12
        assert abs(np.linalg.norm(a - ev[i] * Y[i]) - res[i]) < 1e-11
    eig.close()
    op.close()


@pytest.mark.parametrize("n,nv", [(511, 8), (513, 9), (522240, 17), (522241, 16), (2049, 1), (1048576, 17)])
def test_projection_edges(gpu_ctx, n, nv):
    """c = V^H w and w - V c at the edges of the dots' blocks: elements per thread (2 below 256
    blocks of 2048), groups of 8 vectors, odd counts, a basis just above the Infinity Cache.
    Sums of n products of unit Gaussians: rounding below 1e-13 of ||V_j|| ||w|| (FP64)."""
    import torch
    from paper_0901_3163_amd import deflan
    g = torch.Generator(device="cuda")
    g.manual_seed(n + nv)
    V = torch.view_as_complex(torch.randn((nv, n, 2), generator=g, device="cuda", dtype=torch.float64))
    w = torch.view_as_complex(torch.randn((n, 2), generator=g, device="cuda", dtype=torch.float64))
    c, w2 = deflan.dl_tsk_project(gpu_ctx, V, w, subtract=True)
    ref = (V.conj() * w).sum(1)
    assert float((c - ref).abs().max()) < 1e-13 * 2 * n
    out = w - (ref[:, None] * V).sum(0)
    assert float((w2 - out).abs().max()) < 1e-12 * float(ref.abs().max()) * nv


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (3, 5, 2, 4), (5, 3, 3, 3), (4, 2, 2, 9)])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
def test_layout_conversions_round_trip(gpu_ctx, dims, prec):
    """With kappa = 0 the batch apply is the storage's rounding of its input, whole and in order,
    on lattices whose last tile is ragged, and in both kinds of memory; FP64 is bitwise."""
    import torch
    from paper_0901_3163_amd import deflan
    from lattice_inputs import su3_links
    op = deflan.Operator(gpu_ctx, dims, su3_links(dims, 3), 0.0, deflan.DL_G5M)
    x = np.stack([gaussian_spinor(dims, 50 + i) for i in range(3)])
    y = op.apply_batched(0, {"f64": 0, "f32": 1, "bf16": 2}[prec], x)
    t = torch.view_as_real(torch.from_numpy(x))
    ref = {"f64": t, "f32": t.float().double(), "bf16": t.float().bfloat16().double()}[prec]
    assert np.array_equal(y, torch.view_as_complex(ref).numpy())
    z = op.apply_batched(0, {"f64": 0, "f32": 1, "bf16": 2}[prec], torch.from_numpy(x).cuda())
    assert np.array_equal(z.cpu().numpy(), y)
    op.close()


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (3, 5, 2, 4), (2, 2, 2, 2), (5, 7, 3, 11)])
@pytest.mark.parametrize("order", [0, 1, 2])
def test_hop_per_wave_stencil_bits(gpu_ctx, dims, order, monkeypatch):
    """The one-hop-per-wave stencil (shape 20) adds the same terms in the same order as shape 0: the
    same bits in every storage, M, M^dag and gamma5 M, on ragged tiles and extents of 2."""
    from paper_0901_3163_amd import deflan
    from lattice_inputs import su3_links
    op = deflan.Operator(gpu_ctx, dims, su3_links(dims, 4), 0.131, deflan.DL_G5M)
    psi = np.stack([gaussian_spinor(dims, 70 + i) for i in range(3)])
    for prec in (0, 1, 2):
        for which in (0, 1, 2):
            monkeypatch.setenv("DEFLAN_WILSON_VARIANT", "0,0")
            ref = op.apply_batched(which, prec, psi)
            monkeypatch.setenv("DEFLAN_WILSON_VARIANT", f"20,{order}")
            assert np.array_equal(op.apply_batched(which, prec, psi), ref), (prec, which)
    op.close()


@pytest.mark.parametrize("storage,kind", [("f64", "mdagm"), ("f64", "g5m"), ("f32", "mdagm"), ("bf16", "g5m")])
def test_solves_on_hop_per_wave_stencil(gpu_ctx, storage, kind, monkeypatch):
    """Its fused reductions: a later rhs converges to the oracle's residual on a ragged lattice."""
    from paper_0901_3163_amd import deflan
    from lattice_inputs import su3_links
    dims = (5, 7, 3, 11)
    U = su3_links(dims, 4)
    ora = dirac.WilsonOperator(U, dims, 0.128)
    op = deflan.Operator(gpu_ctx, dims, U, 0.128, deflan.DL_G5M if kind == "g5m" else deflan.DL_MDAGM)
    B = np.stack([gaussian_spinor(dims, 80 + i) for i in range(2)])
    monkeypatch.setenv("DEFLAN_WILSON_VARIANT", "20,0")
    kw = dict() if storage == "f64" else dict(storage={"f32": 1, "bf16": 2}[storage], batched=1)
    X, st, rc = op.solve_next(B, None, 1e-10, **kw)
    assert rc == 0
    for b, x in zip(B, X):
        assert np.linalg.norm(b.ravel() - ora.M(x.ravel())) <= 1.0001e-10 * np.linalg.norm(b)
    op.close()


@pytest.mark.parametrize("dims", [(16, 16, 2, 5), (8, 8, 8, 16), (24, 8, 2, 17), (5, 9, 6, 3), (32, 16, 4, 4),
                                  (256, 2, 2, 2), (7, 11, 2, 9), (3, 5, 7, 6)])
@pytest.mark.parametrize("nrhs", [1, 3])
def test_box_stencil_bits(gpu_ctx, dims, nrhs, monkeypatch):
    """The box stencils (shapes 21 to 26) against shape 0, bit for bit: boxes that fill a block or
    leave threads idle, y and z faces inside and outside the box, whole planes, ragged time chunks,
    an odd number of rhs for two a block, lattices without a box (the last falls back)."""
    from paper_0901_3163_amd import deflan
    from lattice_inputs import su3_links
    op = deflan.Operator(gpu_ctx, dims, su3_links(dims, 4), 0.131, deflan.DL_G5M)
    psi = np.stack([gaussian_spinor(dims, 70 + i) for i in range(nrhs)])
    for prec in (0, 1, 2):
        for which in (0, 1, 2):
            monkeypatch.setenv("DEFLAN_WILSON_VARIANT", "0,0")
            ref = op.apply_batched(which, prec, psi)
            for v in range(21, 27):
                monkeypatch.setenv("DEFLAN_WILSON_VARIANT", f"{v},{(v + which) % 3}")
                assert np.array_equal(op.apply_batched(which, prec, psi), ref), (prec, which, v)
    op.close()


@pytest.mark.parametrize("variant", [21, 23, 24, 26])
@pytest.mark.parametrize("storage,kind", [("f64", "mdagm"), ("f32", "mdagm"), ("bf16", "mdagm"), ("bf16", "g5m")])
def test_solves_on_box_stencil(gpu_ctx, storage, kind, variant, monkeypatch):
    """Their fused reductions and the residual form (FP32 and BF16 reliable updates), with a zero rhs
    whose blocks are masked: every rhs meets the oracle's residual."""
    from paper_0901_3163_amd import deflan
    from lattice_inputs import su3_links
    dims = (8, 12, 4, 6)
    U = su3_links(dims, 4)
    ora = dirac.WilsonOperator(U, dims, 0.128)
    op = deflan.Operator(gpu_ctx, dims, U, 0.128, deflan.DL_G5M if kind == "g5m" else deflan.DL_MDAGM)
    B = np.stack([gaussian_spinor(dims, 80 + i) for i in range(5)])
    B[1] = 0.0
    monkeypatch.setenv("DEFLAN_WILSON_VARIANT", f"{variant},0")
    kw = dict() if storage == "f64" else dict(storage={"f32": 1, "bf16": 2}[storage], batched=1)
    X, st, rc = op.solve_next(B, None, 1e-10, **kw)
    assert rc == 0 and not X[1].any()
    for b, x in zip(B, X):
        assert np.linalg.norm(b.ravel() - ora.M(x.ravel())) <= 1.0001e-10 * np.linalg.norm(b)
    op.close()


# Network kernels at the edges of their split: fewer and more 64-site tiles than the weight gradient's 64
# chunk groups, a last tile that is not full, one field and three.  FP32 sums of 9 * 16 * 3 products over
# three layers against the FP64 oracle: 3 * 432 * 6e-8 = 8e-5, so 1e-4; the same for BF16 mixing against
# the oracle that rounds the same operands.
@pytest.mark.parametrize("dims,nf", [((3, 5, 2, 7), 1), ((6, 5, 13, 11), 3), ((8, 8, 8, 9), 1)])
def test_network_tiles_and_chunks(gpu_ctx, dims, nf):
    from lattice_inputs import su3_links
    from oracle import lowp, ptc
    from paper_0901_3163_amd import deflan
    U = su3_links(dims, 950)
    w = ptc.init_weights(951, scale=1.0)
    ora = dirac.WilsonOperator(U, dims, 0.12)
    M = lambda v: ora.M(v.ravel()).reshape(v.shape)
    Mdag = lambda v: ora.Mdag(v.ravel()).reshape(v.shape)
    B = np.stack([gaussian_spinor(dims, 952 + i) for i in range(nf)])
    X = np.stack([0.4 * gaussian_spinor(dims, 960 + i) for i in range(nf)])
    Ls, Gs = zip(*[ptc.loss_and_grad(U, w, B[i], X[i], dims, M, Mdag) for i in range(nf)])
    op = deflan.Operator(gpu_ctx, dims, U, 0.12, deflan.DL_G5M)
    net = deflan.Net(gpu_ctx, w)
    L, G = net.loss_grad(op, B, X)
    Y, Y16 = net.apply(op, B), net.apply(op, B, prec=deflan.DL_BF16)
    net.close()
    op.close()

    def close(a, b):
        return np.linalg.norm(np.ravel(a) - np.ravel(b)) <= 1e-4 * np.linalg.norm(np.ravel(b))

    assert abs(L - np.mean(Ls)) <= 1e-4 * np.mean(Ls)
    off = 0
    for l in range(3):
        n = 9 * ptc.WIDTHS[l + 1] * ptc.WIDTHS[l]
        assert close(G[off:off + n], np.mean(Gs, axis=0)[off:off + n])
        off += n
    for i in range(nf):
        assert close(Y[i], ptc.forward(U, w, B[i], dims))
        assert close(Y16[i], ptc.forward_lowp(U, w, B[i], dims, lowp.round_bf16))


# The even-odd apply with two right-hand sides a thread (from 512 blocks on) against one a thread: the same
# operations in the same order, so the same bits; an odd number of right-hand sides leaves a half-empty pair.
@pytest.mark.parametrize("which", ["M", "Mdag", "g5M"])
def test_even_odd_two_rhs_a_thread_bits(gpu_ctx, which):
    from lattice_inputs import su3_links
    from paper_0901_3163_amd import deflan
    dims = (16, 16, 16, 16)
    op = deflan.Operator(gpu_ctx, dims, su3_links(dims, 970), 0.12, deflan.DL_G5M | deflan.DL_EVEN_ODD)
    w = {"M": deflan.DL_APPLY_M, "Mdag": deflan.DL_APPLY_MDAG, "g5M": deflan.DL_APPLY_G5M}[which]
    rng = np.random.default_rng(971)
    P = rng.standard_normal((9, np.prod(dims) // 2, 4, 3)) + 1j * rng.standard_normal((9, np.prod(dims) // 2, 4, 3))
    for prec in (deflan.DL_FP32, deflan.DL_BF16):
        got = op.apply_batched(w, prec, P)
        for i in range(len(P)):
            assert np.array_equal(got[i], op.apply_batched(w, prec, P[i:i + 1])[0])
    op.close()


# The FP64 residual in each shape it can take (a forced shape stands for the tuned one): both marching forms
# with each chunk length on a ragged number of slices, and shapes without a residual form.
@pytest.mark.parametrize("variant", [4, 6, 22, 12, 20])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_reliable_updates_in_each_residual_shape(gpu_ctx, storage, variant, monkeypatch):
    from lattice_inputs import su3_links
    from paper_0901_3163_amd import deflan
    dims = (8, 12, 4, 19)
    U = su3_links(dims, 4)
    ora = dirac.WilsonOperator(U, dims, 0.12)
    op = deflan.Operator(gpu_ctx, dims, U, 0.12, deflan.DL_MDAGM)
    B = np.stack([gaussian_spinor(dims, 90 + i) for i in range(3)])
    monkeypatch.setenv("DEFLAN_WILSON_VARIANT", f"{variant},0")
    X, st, rc = op.solve_next(B, None, 1e-10, storage={"f32": 1, "bf16": 2}[storage], batched=1, reliable_every=8)
    assert rc == 0
    for b, x in zip(B, X):
        assert np.linalg.norm(b.ravel() - ora.M(x.ravel())) <= 1.0001e-10 * np.linalg.norm(b)
    op.close()
