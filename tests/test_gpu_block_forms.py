"""Forms of the streaming kernels by the size of their blocks, and the forms for
states larger than the Infinity Cache, against the FP64 oracle or the form that small
grids take."""
import math

import numpy as np
import pytest
import torch

from gpu_common import Q, make_pair, rel_err, require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


@pytest.fixture(scope="module")
def oracle():
    from oracle import oracle as O
    return O


# blocks of 64, 128, 192 and 256 threads (rows of 32 to 36 nodes, their cells along y
# dealt 2, 4, 6 and 7 to a block), the last one ragged along y
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_el,p", [((8, 13, 3), 4), ((8, 4, 3), 4), ((8, 6, 2), 4), ((8, 7, 2), 4), ((12, 5, 2), 3),
                                    ((6, 3, 2), 6), ((10, 1, 4), 6), ((7, 11, 2), 5), ((7, 3, 3), 5), ((32, 3, 5), 1)])
def test_streaming_by_block_size(oracle, precision, n_el, p):
    """S against the oracle (1e-12, FP32 1e-5: the repository's bars), S^T as its
    adjoint per velocity."""
    ctx, cfg = make_pair(oracle, n_el, p, 0.06, 0.01, precision=precision)
    rng = np.random.default_rng(17)
    x, y = (rng.normal(size=(2, Q, ctx.nodes)).astype(np.float32).astype(np.float64) for _ in range(2))
    print("block form", precision, n_el, p, flush=True)
    F, G = to_np(ctx.stream(to_dev(ctx, x[0], x[1])))
    f, g = oracle.stream(cfg, x[0], x[1])
    tol = 1e-5 if precision else 1e-12
    assert rel_err(F, f) < tol and rel_err(G, g) < tol
    st = np.stack(to_np(ctx.stream(to_dev(ctx, y[0], y[1]), transpose=True)))
    fg = np.stack([f, g])
    lhs, rhs = (fg * y).sum(-1), (x * st).sum(-1)
    assert np.all(np.abs(lhs - rhs) <= tol * (np.abs(fg * y).sum(-1) + np.abs(x * st).sum(-1)))


# order 6 with one block per plane (marched) and two
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_el", [(1, 1, 1), (2, 3, 1), (7, 4, 1), (7, 5, 1), (2, 3, 2)])
def test_graded_streaming_of_few_cells(oracle, precision, n_el):
    """Graded S of order 6 against the oracle (1e-12, FP32 1e-5)."""
    from paper_2012_05537_amd.sllbm import SLLBM
    rng = np.random.default_rng(sum(n_el))
    widths = []
    for n in n_el:
        w = 1.0 + 0.4 * rng.uniform(-1.0, 1.0, n)
        widths.append(w * (2 * np.pi / w.sum()))
    ctx = SLLBM(n_el, 6, 0.2, 0.01, precision=precision)
    ctx.set_mesh(*widths)
    cfg = oracle.make_cfg(n_el, 6, 0.2, 0.01, widths=widths)
    x = rng.normal(size=(2, Q, ctx.nodes)).astype(np.float32).astype(np.float64)
    print("graded, few cells", precision, n_el, flush=True)
    F, G = to_np(ctx.stream(to_dev(ctx, x[0], x[1])))
    f, g = oracle.stream(cfg, x[0], x[1])
    tol = 1e-5 if precision else 1e-12
    assert rel_err(F, f) < tol and rel_err(G, g) < tol


# states larger than the Infinity Cache, x rows of whole cache lines: non-temporal
# stores, at every order in both precisions, blocks of 64 to 1024 threads
LARGE = [((80, 70, 70), 1, 0), ((40, 36, 37), 2, 0), ((16, 32, 31), 3, 0), ((20, 20, 20), 4, 0), ((8, 13, 57), 4, 0),
         ((8, 4, 183), 4, 0), ((16, 14, 14), 5, 0), ((16, 12, 12), 6, 0), ((96, 90, 87), 1, 1), ((48, 46, 45), 2, 1),
         ((32, 30, 31), 3, 1), ((24, 23, 24), 4, 1), ((8, 13, 120), 4, 1), ((32, 14, 14), 5, 1), ((16, 16, 15), 6, 1),
         ((320, 40, 32), 1, 0), ((640, 25, 25), 1, 0), ((160, 20, 20), 2, 0), ((512, 10, 10), 2, 0), ((128, 11, 12), 3, 0),
         ((96, 8, 8), 4, 0), ((160, 7, 7), 4, 0), ((256, 5, 5), 4, 0), ((224, 12, 12), 3, 1), ((192, 9, 9), 4, 1),
         ((256, 7, 7), 4, 1)]


# and of others: whole rows of 260 to 500 nodes with idle lanes, longer rows in tiles, and
# rows of order 5 in tiles
OTHER = [((65, 10, 10), 4, 0), ((125, 10, 10), 4, 1), ((107, 12, 12), 3, 0), ((150, 7, 7), 4, 0), ((300, 20, 20), 2, 1),
         ((64, 8, 8), 5, 0)]


@pytest.mark.parametrize("n_el,p,precision", LARGE + OTHER)
def test_large_grid_streaming(oracle, n_el, p, precision):
    """Two z-planes of S against the oracle (1e-12, FP32 1e-5), S^T by <S x, y> = <x, S^T y>
    per population and velocity, relative to the sums of the terms' magnitudes."""
    dt = 3.0 * (2 * math.pi / (max(n_el) * p)) / math.sqrt(15.0)
    ctx, cfg = make_pair(oracle, n_el, p, dt, 1e-3, precision=precision)
    elem = 4 if precision else 8
    assert 90 * ctx.nodes * elem > 256 << 20
    assert n_el[0] * p * elem % 128 == 0 or (n_el, p, precision) in OTHER
    print("large grid", precision, n_el, p, flush=True)
    gen = torch.Generator(device=ctx.device).manual_seed(p)
    x, y = (torch.randn((2, Q, ctx.nodes), generator=gen, device=ctx.device, dtype=ctx.dtype) for _ in range(2))
    s = ctx.stream(x)
    f0, g0 = to_np(x)
    plane = ctx.shape[1] * ctx.shape[2]
    tol = 1e-5 if precision else 1e-12
    for z in (0, ctx.shape[0] // 2 + 1):
        fs, gs = oracle.stream_at_nodes(cfg, f0, g0, z * plane + np.arange(plane))
        F, G = (v[:, z * plane:(z + 1) * plane].double().cpu().numpy().T for v in s)
        assert np.max(np.abs(F - fs)) / np.abs(fs).max() < tol and np.max(np.abs(G - gs)) / np.abs(gs).max() < tol
    st = ctx.stream(y, transpose=True)
    lhs, rhs = (s.double() * y.double()), (x.double() * st.double())
    scale = lhs.abs().sum(2) + rhs.abs().sum(2)
    assert float(((lhs.sum(2) - rhs.sum(2)).abs() / scale).max()) < tol
    ctx.close()


# staged up to one block of 64 nodes per CU, in registers beyond, there with
# non-temporal accesses above 256 MiB (80^3 nodes)
@pytest.mark.parametrize("n_el,p", [((32, 32, 16), 1), ((114, 48, 3), 1), ((20, 20, 20), 4)])
def test_fp64_reverse_step_forms_agree(n_el, p):
    """FP64 reverse step of copies of a 32-node grid's state and adjoint.  Cells of
    length 1e14 and more leave every node on itself, so that the step is the
    collision's VJP: equal node by node to rounding (4e-13 of the largest value), and
    dL/dmu the number of copies times the small grid's (1e-10)."""
    from paper_2012_05537_amd.sllbm import SLLBM
    small, large = SLLBM((4, 4, 2), 1, 0.05, 0.02, length=1e16), SLLBM(n_el, p, 0.05, 0.02, length=1e16)
    assert large.nodes % 32 == 0 and (p == 1 or 90 * large.nodes * 8 > 256 << 20)
    gen = torch.Generator(device=small.device).manual_seed(3)
    rnd = lambda *s: torch.randn(s, generator=gen, device=small.device, dtype=torch.float64)
    small.init_equilibrium(1 + 0.1 * rnd(32), 0.2 * rnd(3, 32), 1 + 0.05 * rnd(32))
    x = small.get_state() * (1 + 0.02 * rnd(2, Q, 32))
    lam = rnd(2, Q, 32) + 0.5
    print("FP64 reverse step", n_el, flush=True)
    dmu = torch.zeros(2, dtype=torch.float64, device=small.device)
    want = small.adjoint_step(x, lam, dmu=dmu[:1])
    reps = large.nodes // 32
    got = large.adjoint_step(x.repeat(1, 1, reps), lam.repeat(1, 1, reps), dmu=dmu[1:])
    assert float((got.view(2, Q, reps, 32) - want[:, :, None]).abs().max() / want.abs().max()) <= 4e-13
    assert float(dmu[1]) == pytest.approx(reps * float(dmu[0]), rel=1e-10)


# FP64 collision: staged up to one block of 64 nodes per CU, in registers while two
# states fit the Infinity Cache (186,413 nodes), staged beyond
@pytest.mark.parametrize("n_el", [(32, 32, 16), (114, 48, 3), (64, 56, 52), (74, 60, 42)])
def test_fp64_collision_forms_agree(oracle, n_el):
    """Collision of a grid of copies of a small one, whose collision is checked against
    the oracle (1e-12, the repository's bar): equal to rounding (1e-13)."""
    ctx, _ = make_pair(oracle, n_el, 1, 0.05, 0.02)
    small, cfg = make_pair(oracle, (4, 4, 2), 1, 0.05, 0.02)
    rng = np.random.default_rng(23)
    f, g = oracle.init_equilibrium(cfg, 1 + 0.1 * rng.normal(size=32), 0.2 * rng.normal(size=(3, 32)),
                                   1 + 0.05 * rng.normal(size=32))
    f, g = f * (1 + 0.02 * rng.normal(size=f.shape)), g * (1 + 0.02 * rng.normal(size=g.shape))
    x = to_dev(small, f, g)
    print("FP64 collision form", n_el, flush=True)
    want = small.collide(x.clone())
    fo, go = oracle.collide(cfg, f, g)
    F, G = to_np(want)
    assert rel_err(F, fo) < 1e-12 and rel_err(G, go) < 1e-12
    reps = -(-ctx.nodes // 32)
    got = ctx.collide(x.repeat(1, 1, reps)[:, :, :ctx.nodes].contiguous())
    assert float((got - want.repeat(1, 1, reps)[:, :, :ctx.nodes]).abs().max() / want.abs().max()) <= 1e-13
