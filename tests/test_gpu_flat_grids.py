"""One- and two-dimensional grids (one cell along y or z): the stage kernel variant that
leaves out the fluxes of those axes gives bit for bit what the general kernel gives.

The general kernel runs such grids through rhs_flags (limiters on: its variant records
every face) and in batches of two members; both are compared with the single-problem
calls, which take the reduced kernel.
"""
import numpy as np
import pytest
import torch

from paper_2402_05193_amd import solver as S

pytestmark = pytest.mark.gpu

SHAPES = [(33, 1, 1), (1, 1, 21), (1, 19, 1), (35, 18, 1), (17, 1, 20), (1, 16, 3), (5, 1, 1)]
PERIODIC, OPEN = (S.PERIODIC,) * 6, (S.ZERO_GRADIENT,) * 6


def state(cfg, seed):
    rng = np.random.default_rng(seed)
    W = 1.0 + 0.2 * rng.random(cfg.shape)
    v = 2 if cfg.model == S.DIM else 1
    W[v:v + 3] = 0.3 * rng.standard_normal(W[v:v + 3].shape)
    if cfg.model == S.DIM:
        W[6] = rng.choice([1e-8, 0.3, 0.7, 1 - 1e-8], size=W[6].shape)
        W[0], W[1] = W[6] * W[0], (1 - W[6]) * W[1]
    U = S.empty_state(cfg)
    return S.prim_to_cons(cfg, torch.from_numpy(W).to("cuda", cfg.torch_dtype).contiguous(), U)


def config(shape, model, dtype, bc, positivity, thinc=0):
    return S.Config(nx=shape[0], ny=shape[1], nz=shape[2], dx=0.1, dy=0.12, dz=0.09, model=model, dtype=dtype, bc=bc,
                    positivity=positivity, mu=1e-2 if model == S.NS else 0.0, gamma2=1.66, thinc=thinc)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("model,thinc", [(S.EULER, 0), (S.NS, 0), (S.DIM, 0), (S.DIM, 1)])
@pytest.mark.parametrize("dtype", [S.F64, S.F32])
@pytest.mark.parametrize("bc", [PERIODIC, OPEN])
def test_flat_rhs_equals_the_recording_kernel(shape, model, thinc, dtype, bc):
    cfg = config(shape, model, dtype, bc, 1, thinc)
    U = state(cfg, 3)
    R, _ = S.rhs_flags(cfg, U, torch.empty_like(U), 1e-3)
    got = S.rhs(cfg, U, torch.full_like(U, float("nan")), 1e-3)
    assert torch.isfinite(got).all()
    assert torch.equal(got, R)


@pytest.mark.parametrize("shape", SHAPES[:5])
@pytest.mark.parametrize("model", [S.EULER, S.NS, S.DIM])
@pytest.mark.parametrize("positivity", [0, 1])
def test_flat_advance_equals_the_batched_kernel(shape, model, positivity):
    members, alone = [], []
    for k in range(2):
        cfg = config(shape, model, S.F64, OPEN if k else PERIODIC, positivity)
        U, ws = state(cfg, 10 + k), S.workspace(cfg)
        V = U.clone()
        S.advance(cfg, V, 3, 0.0, ws)
        alone.append(V)
        members.append((cfg, U, S.workspace(cfg)))
    b = S.Batch(2)
    b.set(members, fresh=[1, 1])
    b.step(3)
    torch.cuda.synchronize()
    for (_, U, _), V in zip(members, alone):
        assert torch.equal(U, V)
    b.close()


@pytest.mark.parametrize("shape", [(9, 1, 1), (9, 8, 1)])
def test_flat_inadmissible_cell_gives_nan(shape):
    """A cell whose own flux is not a number (negative pressure, limiters off) has no finite
    right-hand side, as with every face evaluated."""
    cfg = config(shape, S.EULER, S.F64, PERIODIC, 0)
    U = state(cfg, 5)
    U[4, 0, 0, 4] = -1.0
    R = S.rhs(cfg, U, torch.empty_like(U))
    assert torch.isnan(R[:, 0, 0, 4]).all()


@pytest.mark.parametrize("shape", [(9, 1, 1), (9, 8, 1), (9, 1, 6)])
@pytest.mark.parametrize("law", [1, 2])
def test_flat_viscosity_law_below_zero_temperature(shape, law):
    """A cell in tension (p < 0 < p + p_inf) has a convective flux but no viscosity at its
    temperature p / rho: not a number where the recording kernel has none, else equal."""
    cfg = config(shape, S.NS, S.F64, PERIODIC, 1)
    cfg.pinf1, cfg.visc_law, cfg.T_ref, cfg.sutherland = 10.0, law, 0.9, 0.35
    U = state(cfg, 8)
    W = S.cons_to_prim(cfg, U, torch.empty_like(U))
    W[4, 0, 0, 4] = -0.5
    U = S.prim_to_cons(cfg, W, U)
    R, _ = S.rhs_flags(cfg, U, torch.empty_like(U), 1e-3)
    got = S.rhs(cfg, U, torch.empty_like(U), 1e-3)
    assert torch.isnan(R[1:, 0, 0, 4]).all() and torch.isfinite(R[:, 0, 0, 0]).all()
    assert torch.equal(got.nan_to_num(nan=1e30), R.nan_to_num(nan=1e30))


@pytest.mark.parametrize("model", [S.EULER, S.DIM])
@pytest.mark.parametrize("axis", [1, 2])
@pytest.mark.parametrize("scale", [1.0, 1e13])
def test_flat_flux_beyond_the_range(model, axis, scale):
    """Uniform flow along an axis of one cell: finite, or (FP32, energy flux of 1e41) not a
    number, as the recording kernel has it."""
    cfg = config((9, 1, 1), model, S.F32, PERIODIC, 1)
    v = 2 if model == S.DIM else 1
    W = torch.ones(cfg.shape, device="cuda")
    W[:v] = 1.0 / v
    W[v:v + 3] = 0.0
    W[v + axis] = scale
    W[v + 3] = scale * scale * 100.0
    if model == S.DIM:
        W[6] = 0.5
    U = S.prim_to_cons(cfg, W, S.empty_state(cfg))
    assert torch.isfinite(U).all()
    R, _ = S.rhs_flags(cfg, U, torch.empty_like(U), 1e-20)
    got = S.rhs(cfg, U, torch.empty_like(U), 1e-20)
    assert torch.isfinite(R[v + 3]).all() == (scale == 1.0)
    assert torch.equal(torch.isnan(got), torch.isnan(R))
    if scale == 1.0:
        assert torch.equal(got, R)


def walls(shape):
    """Symmetry planes on the axes that can hold them, open boundaries on the others."""
    return tuple(b for n in shape for b in ((S.SYMMETRY, S.ZERO_GRADIENT) if n >= 3 else OPEN[:2]))


VARIANTS = [dict(model=S.EULER), dict(model=S.NS, visc_law=1, T_ref=0.9), dict(model=S.NS, visc_law=2, sutherland=0.35),
            dict(model=S.DIM), dict(model=S.DIM, thinc=1)]


def variant(shape, dtype, bc, positivity, kw):
    cfg = config(shape, kw["model"], dtype, bc, positivity)
    for k, v in kw.items():
        setattr(cfg, k, v)
    return cfg


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kw", VARIANTS)
@pytest.mark.parametrize("dtype", [S.F64, S.F32])
def test_flat_rhs_with_walls_and_viscosity_laws(shape, kw, dtype):
    cfg = variant(shape, dtype, walls(shape), 1, kw)
    U = state(cfg, 4)
    R, _ = S.rhs_flags(cfg, U, torch.empty_like(U), 1e-3)
    got = S.rhs(cfg, U, torch.full_like(U, float("nan")), 1e-3)
    assert torch.isfinite(got).all()
    assert torch.equal(got, R)


@pytest.mark.parametrize("shape", SHAPES[:5])
@pytest.mark.parametrize("kw", VARIANTS)
def test_flat_advance_with_walls_and_viscosity_laws(shape, kw):
    """The stages with their CFL reduction, against the batched kernel."""
    members, alone = [], []
    for k in range(2):
        cfg = variant(shape, S.F64, walls(shape) if k else PERIODIC, 1, kw)
        U, ws = state(cfg, 20 + k), S.workspace(cfg)
        V = U.clone()
        alone.append((V, S.advance(cfg, V, 3, 0.0, ws, t=0.0)))
        members.append((cfg, U, S.workspace(cfg)))
    b = S.Batch(2)
    b.set(members, fresh=[1, 1])
    b.step(3)
    torch.cuda.synchronize()
    for (cfg, U, ws), (V, t) in zip(members, alone):
        assert torch.isfinite(U).all() and torch.equal(U, V)
        assert S.workspace_time(cfg, ws) == t
    b.close()
