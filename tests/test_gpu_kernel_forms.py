"""The forms a kernel has for different sizes, alignments and grids, at the
sizes where they can go wrong (remainders of tiles and blocks, smallest grids,
unaligned buffers), against each other or the FP64 oracle."""

import numpy as np
import pytest
import torch

from gpu_common import Q, make_pair, rel_err, require_gpu, to_dev, to_np
from paper_2012_05537_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


@pytest.fixture(scope="module")
def oracle():
    from oracle import oracle as O
    return O


def _noisy(oracle, cfg, seed, Ma=0.7):
    f, g = oracle.init_equilibrium(cfg, *inputs.tgv_fields(*oracle.node_coords(cfg), Ma, 1.4))
    rng = np.random.default_rng(seed)
    return f * (1 + 0.03 * rng.normal(size=f.shape)), g * (1 + 0.03 * rng.normal(size=g.shape))


# nodes: 1, 27 (odd: register form), 64 (one FP64 block), 130 and 132 (ragged
# blocks; 130 is no multiple of 4: register form in FP32), 2000
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_el,p", [((1, 1, 1), 1), ((1, 1, 1), 3), ((2, 2, 2), 2), ((13, 5, 2), 1), ((11, 4, 3), 1),
                                    ((5, 2, 2), 5)])
def test_collision_vjp_forms_agree(oracle, precision, n_el, p):
    """alpha staged in LDS (aligned buffers) and in registers (a lambda buffer
    one element past a 16-byte boundary) run the same arithmetic: equal bits,
    and the derivative along a random direction matches the complex step of
    the oracle's collision (1e-12 per unit of sum |terms| in FP64; in FP32 the
    outputs are rounded once, 2^-23 of the same sum)."""
    ctx, cfg = make_pair(oracle, n_el, p, 0.05, 0.02, precision=precision)
    f, g = _noisy(oracle, cfg, 3)
    if precision:
        f, g = f.astype(np.float32).astype(np.float64), g.astype(np.float32).astype(np.float64)
    x = to_dev(ctx, f, g)
    rng = np.random.default_rng(4)
    lam = torch.from_numpy(rng.normal(size=x.shape)).to(ctx.device, ctx.dtype)
    n = x.numel()
    flat = torch.zeros(n + 1, dtype=ctx.dtype, device=ctx.device)
    off = flat[1:].view(x.shape)
    al = ctx.empty_state()
    dmu = torch.zeros(2, dtype=torch.float64, device=ctx.device)
    print("vjp forms", precision, n_el, p, flush=True)
    ctx.adjoint_step(x, lam, al, dmu[:1])
    ctx.adjoint_step(x, lam, off, dmu[1:])
    assert torch.equal(al, off)
    assert float(dmu[0]) == pytest.approx(float(dmu[1]), rel=1e-9, abs=1e-12 * float(lam.abs().sum()))
    # <lam_out, d> = <S^T lam, J_C d>
    d = rng.normal(size=(2,) + f.shape)
    h = 1e-30
    fc, gc = oracle.collide(cfg, f + 1j * h * d[0], g + 1j * h * d[1])
    st = to_np(ctx.stream(lam, transpose=True))
    L = to_np(al)
    terms = np.abs(st[0] * fc.imag / h).sum() + np.abs(st[1] * gc.imag / h).sum() + np.abs(L[0] * d[0]).sum() + \
        np.abs(L[1] * d[1]).sum()
    ref = (st[0] * fc.imag / h).sum() + (st[1] * gc.imag / h).sum()
    got = (L[0] * d[0]).sum() + (L[1] * d[1]).sum()
    assert abs(got - ref) <= (2.0 ** -23 if precision else 1e-12) * terms


def _displacement(ctx, a):
    xs, ys, zs = (c.numpy() for c in ctx.node_coords())
    X, Y, Z = inputs.mesh(xs, ys, zs)
    return a * np.stack([np.sin(X + Y) + 0.3 * np.cos(2 * Z), np.cos(Y + Z), np.sin(Z - X)])


# orders below and from the change of kernel on; one-cell axes, a row of cells
# longer than a run (19 cells: two runs), shifts of several cells, a ragged row
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_el,p,dt", [((1, 2, 1), 3, 0.3), ((19, 2, 2), 3, 0.05), ((5, 4, 3), 3, 0.4), ((17, 3, 1), 4, 0.02),
                                       ((3, 3, 4), 4, 0.3), ((9, 2, 2), 5, 0.1), ((2, 3, 7), 6, 0.1), ((4, 3, 5), 2, 0.2)])
def test_distorted_streaming_by_cell(oracle, precision, n_el, p, dt):
    """Streaming on distorted cells against the oracle (1e-12, FP32 1e-5, the
    repository's bars), and its transpose as the adjoint of it."""
    from paper_2012_05537_amd.sllbm import SLLBM
    ctx = SLLBM(n_el, p, dt, 0.01, precision=precision)
    d = _displacement(ctx, 0.02)
    ctx.set_displacement(d)
    cfg = oracle.make_cfg(n_el, p, dt, 0.01, disp=d)
    rng = np.random.default_rng(8)
    x = rng.normal(size=(2, Q, ctx.nodes)).astype(np.float32).astype(np.float64)
    y = rng.normal(size=x.shape).astype(np.float32).astype(np.float64)
    print("distorted streaming", precision, n_el, p, flush=True)
    S = to_np(ctx.stream(to_dev(ctx, x[0], x[1])))
    f, g = oracle.stream(cfg, x[0], x[1])
    tol = 1e-5 if precision else 1e-12
    assert rel_err(S[0], f) < tol and rel_err(S[1], g) < tol
    st = to_np(ctx.stream(to_dev(ctx, y[0], y[1]), transpose=True))
    a, b = (f * y[0]).sum() + (g * y[1]).sum(), (x[0] * st[0]).sum() + (x[1] * st[1]).sum()
    scale = np.abs(f * y[0]).sum() + np.abs(g * y[1]).sum()
    assert abs(a - b) <= tol * scale


# whole rows up to 256 nodes and split ones beyond (a ragged last tile, two
# tiles of one cell row), one-cell axes, ragged blocks along y, blocks of one
# and of several cells along z, shifts of several cells
STREAM_FORMS = [((1, 1, 1), 1, 0.9), ((256, 2, 3), 1, 0.02), ((257, 1, 2), 1, 0.05), ((3, 300, 2), 1, 0.3),
                ((5, 4, 70), 1, 0.1), ((129, 3, 5), 2, 0.02), ((2, 2, 9), 2, 0.8), ((43, 7, 3), 3, 0.05),
                ((86, 2, 1), 3, 0.03), ((64, 1, 2), 4, 0.01), ((65, 3, 6), 4, 0.02), ((1, 1, 9), 4, 0.7),
                ((51, 6, 2), 5, 0.03), ((52, 1, 5), 5, 0.02), ((43, 2, 1), 6, 0.03), ((2, 3, 9), 6, 1.1)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_el,p,dt", STREAM_FORMS)
def test_streaming_by_source_cell(oracle, precision, n_el, p, dt):
    """Equal-cell streaming against the oracle (1e-12, FP32 1e-5: the
    repository's bars), from and into buffers at any element offset."""
    ctx, cfg = make_pair(oracle, n_el, p, dt, 0.01, precision=precision)
    rng = np.random.default_rng(11)
    x = rng.normal(size=(2, Q, ctx.nodes)).astype(np.float32).astype(np.float64)
    xd = to_dev(ctx, x[0], x[1])
    print("streaming form", precision, n_el, p, flush=True)
    out = ctx.stream(xd)
    flat = torch.zeros(2 * xd.numel() + 3, dtype=ctx.dtype, device=ctx.device)
    a, b = flat[1:1 + xd.numel()].view(xd.shape), flat[-xd.numel() - 1:-1].view(xd.shape)
    a.copy_(xd)
    assert torch.equal(ctx.stream(a, out=b), out)
    F, G = to_np(out)
    f, g = oracle.stream(cfg, x[0], x[1])
    tol = 1e-5 if precision else 1e-12
    assert rel_err(F, f) < tol and rel_err(G, g) < tol
    # and the transpose as the adjoint of it, per velocity
    y = rng.normal(size=x.shape).astype(np.float32).astype(np.float64)
    yd = to_dev(ctx, y[0], y[1])
    st = ctx.stream(yd, transpose=True)
    a.copy_(yd)
    assert torch.equal(ctx.stream(a, transpose=True, out=b), st)
    st = st.cpu().double().numpy()
    fg = np.stack([f, g])
    lhs, rhs = (fg * y).sum(-1), (x * st).sum(-1)
    assert np.all(np.abs(lhs - rhs) <= tol * (np.abs(fg * y).sum(-1) + np.abs(x * st).sum(-1)))


# rows of one to four waves with and without idle lanes, a row too long for a
# block and orders that are marched, blocks ragged along y, blocks of one and of
# several cells along z with a remainder, one-cell axes, shifts of several
# cells, and a grading with cells that nothing departs into and cells with more
# than P + 3 readers
GRADED_FORMS = [((16, 5, 6), 4, 0.05, 0.4), ((17, 3, 9), 4, 0.05, 0.4), ((43, 2, 3), 3, 0.03, 0.4),
                ((64, 1, 2), 4, 0.02, 0.4), ((65, 2, 2), 4, 0.02, 0.4), ((33, 5, 2), 6, 0.04, 0.4),
                ((3, 9, 40), 2, 0.1, 0.4), ((1, 1, 5), 3, 0.9, 0.4), ((5, 7, 1), 5, 0.3, 0.4),
                ((4, 6, 5), 6, 1.1, 0.3), ((9, 8, 7), 3, 0.2, 0.9), ((9, 4, 3), 1, 0.2, 0.4)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_el,p,dt,amp", GRADED_FORMS)
def test_graded_streaming_by_source_cell(oracle, precision, n_el, p, dt, amp):
    """Streaming on graded cells against the oracle (1e-12, FP32 1e-5: the
    repository's bars) and its transpose as the adjoint of it, per velocity."""
    from paper_2012_05537_amd.sllbm import SLLBM
    rng = np.random.default_rng(sum(n_el) + p)
    widths = []
    for n in n_el:
        w = 1.0 + amp * rng.uniform(-1.0, 1.0, n)
        widths.append(w * (2 * np.pi / w.sum()))
    ctx = SLLBM(n_el, p, dt, 0.01, precision=precision)
    ctx.set_mesh(*widths)
    cfg = oracle.make_cfg(n_el, p, dt, 0.01, widths=widths)
    x = rng.normal(size=(2, Q, ctx.nodes)).astype(np.float32).astype(np.float64)
    y = rng.normal(size=x.shape).astype(np.float32).astype(np.float64)
    print("graded form", precision, n_el, p, flush=True)
    F, G = to_np(ctx.stream(to_dev(ctx, x[0], x[1])))
    f, g = oracle.stream(cfg, x[0], x[1])
    tol = 1e-5 if precision else 1e-12
    assert rel_err(F, f) < tol and rel_err(G, g) < tol
    st = np.stack(to_np(ctx.stream(to_dev(ctx, y[0], y[1]), transpose=True)))
    fg = np.stack([f, g])
    lhs, rhs = (fg * y).sum(-1), (x * st).sum(-1)
    assert np.all(np.abs(lhs - rhs) <= tol * (np.abs(fg * y).sum(-1) + np.abs(x * st).sum(-1)))


# rows that are not 16-byte aligned, staged by words: 41 x 41 x 41 (FP32; a last block
# of one node) and 73 x 73 x 73 nodes (FP64, larger than the Infinity Cache; of
# 9 nodes)
@pytest.mark.parametrize("precision,n", [(1, 41), (0, 73)])
def test_collision_staged_by_words(oracle, precision, n):
    """Collision and its VJP of an odd grid against the same nodes in a small
    grid, whose collision is another kernel form: equal to rounding (the moments
    are summed in the same order: 1e-13 in FP64, one rounding in FP32)."""
    ctx, _ = make_pair(oracle, (n, n, n), 1, 0.05, 0.02, precision=precision)
    small, cfg = make_pair(oracle, (3, 3, 3), 1, 0.05, 0.02, precision=precision)
    f, g = _noisy(oracle, cfg, 5)
    s = to_dev(small, f, g)
    k = small.nodes
    reps = -(-ctx.nodes // k)
    x = s.repeat(1, 1, reps)[:, :, :ctx.nodes].contiguous()
    print("staged by words", precision, n, flush=True)
    want = small.collide(s.clone()).repeat(1, 1, reps)[:, :, :ctx.nodes]
    got = ctx.collide(x.clone())
    tol = 2.0 ** -23 if precision else 1e-13
    assert float(((got - want).abs() / want.abs().amax()).max()) <= tol
    lam = torch.from_numpy(np.random.default_rng(6).normal(size=s.shape)).to(ctx.device, ctx.dtype)
    lam = lam.repeat(1, 1, reps)[:, :, :ctx.nodes].contiguous()
    out = ctx.adjoint_step(x, lam)
    # the same VJP of the streamed adjoint, node by node, in the small grid's form
    st = ctx.stream(lam, transpose=True)
    i0 = (ctx.nodes // k - 2) * k
    y = torch.empty_like(s)
    dmu = torch.zeros(1, dtype=torch.float64, device=ctx.device)
    small_out = _vjp_of(small, s, st[:, :, i0:i0 + k].contiguous(), y, dmu)
    sel = out[:, :, i0:i0 + k]
    assert float((sel - small_out).abs().max() / small_out.abs().max()) <= 4 * tol


def _vjp_of(ctx, x, alpha, out, dmu):
    """Collision VJP alone: the transposed streaming undone by a zero shift (dt
    tiny leaves every node on itself), so that adjoint_step is the VJP."""
    from paper_2012_05537_amd.sllbm import SLLBM
    c = ctx.cfg
    still = SLLBM(tuple(c.n_el), c.order, c.dt, c.mu_inf, precision=c.precision,
                  length=tuple(1e16 for _ in range(3)))
    return still.adjoint_step(x, alpha, out, dmu).clone()


# the copy kernel (64^3 nodes, FP64, and 97 x 97 x 65 FP32: 8 bytes past whole
# vectors) and hipMemcpyAsync (a buffer one element off)
@pytest.mark.parametrize("n_el,precision", [((64, 64, 64), 0), ((97, 97, 65), 1)])
def test_large_state_copies(n_el, precision):
    from paper_2012_05537_amd.sllbm import SLLBM
    ctx = SLLBM(n_el, 1, 0.01, 0.01, precision=precision)
    x = torch.rand((2, Q, ctx.nodes), dtype=ctx.dtype, device=ctx.device)
    guard = torch.zeros(x.numel() + 8, dtype=ctx.dtype, device=ctx.device)
    print("state copies", n_el, precision, flush=True)
    ctx.set_state(x)
    for off in (4, 3):
        out = guard[off:off + x.numel()].view(x.shape)
        ctx.get_state(out)
        assert torch.equal(out, x)
        assert not guard[:off].any() and not guard[off + x.numel():].any()
        guard.zero_()


# whole rows up to 256 nodes (512 beyond 65536 nodes in all) and split ones, a
# ragged last tile, groups of cells along y with a remainder, one-cell axes,
# shifts of several cells
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_el,p,shift", [((1, 1), 4, 0.7), ((64, 2), 4, 0.3), ((65, 3), 4, 2.3), ((512, 130), 1, 0.4),
                                          ((513, 130), 1, 1.7), ((129, 5), 2, 0.2), ((2, 41), 2, 3.1), ((13, 11), 3, 0.9),
                                          ((86, 3), 3, 0.1), ((103, 2), 5, 0.6), ((3, 70), 6, 1.2), ((43, 2), 6, 0.1)])
def test_streaming_2d_by_source_cell(precision, n_el, p, shift):
    """Two-dimensional streaming against its oracle (1e-12, FP32 1e-5: the
    repository's bars); shift: largest displacement in cells along x."""
    from oracle import oracle2d as O2
    from paper_2012_05537_amd.sllbm import CONSTANT, D2Q19, SLLBM
    dt = shift / n_el[0] / 3.5
    length = (1.0, 0.7 * n_el[1] / n_el[0])
    ctx = SLLBM(n_el, p, dt, 1e-3, length=length, viscosity_law=CONSTANT, precision=precision, velocity_set=D2Q19)
    cfg = O2.make_cfg(n_el, p, dt, 1e-3, length=length, viscosity_law=O2.CONSTANT)
    x = np.random.default_rng(9).normal(size=(2, 19, ctx.nodes)).astype(np.float32).astype(np.float64)
    print("2-D streaming form", precision, n_el, p, flush=True)
    F, G = to_np(ctx.stream(to_dev(ctx, x[0], x[1])))
    f, g = O2.stream(cfg, x[0], x[1])
    tol = 1e-5 if precision else 1e-12
    assert rel_err(F, f) < tol and rel_err(G, g) < tol
