"""The order in which a single-problem launch gives its workgroups to tiles and z chunks
(a contiguous range per XCD, whatever the count modulo eight) reaches every cell: the
results are bit for bit those of the batched kernel, which keeps the plain order.
"""
import numpy as np
import pytest
import torch

from paper_2402_05193_amd import solver as S

pytestmark = pytest.mark.gpu


# small grids take z chunks of one plane: ceil(nx/16) ceil(ny/16) nz workgroups
@pytest.mark.parametrize("shape", [(16, 16, 2), (9, 20, 5), (16, 16, 9), (33, 16, 5), (33, 17, 3), (50, 35, 7), (64, 48, 13)])
@pytest.mark.parametrize("model,dtype", [(S.EULER, S.F64), (S.NS, S.F64), (S.NS, S.F32), (S.DIM, S.F64)])
def test_every_cell_is_reached(shape, model, dtype):
    members, alone = [], []
    for k in range(2):
        cfg = S.Config(nx=shape[0], ny=shape[1], nz=shape[2], dx=0.1, dy=0.12, dz=0.09, model=model, dtype=dtype,
                       bc=(S.PERIODIC,) * 6 if k else (S.ZERO_GRADIENT,) * 6, mu=1e-2 if model == S.NS else 0.0,
                       gamma2=1.66)
        rng = np.random.default_rng(7 + k)
        W = 1.0 + 0.1 * rng.random(cfg.shape)
        if model == S.DIM:
            W[6] = 0.2 + 0.6 * rng.random(W[6].shape)
        U = S.prim_to_cons(cfg, torch.from_numpy(W).to("cuda", cfg.torch_dtype).contiguous(), S.empty_state(cfg))
        V = U.clone()
        S.advance(cfg, V, 2, 0.0, S.workspace(cfg))
        assert torch.isfinite(V).all()
        alone.append(V)
        members.append((cfg, U, S.workspace(cfg)))
    b = S.Batch(2)
    b.set(members, fresh=[1, 1])
    b.step(2)
    torch.cuda.synchronize()
    for (_, U, _), V in zip(members, alone):
        assert torch.equal(U, V)
    b.close()


def test_long_line():
    """A line of so many cells along z that chunks of the usual length would exceed the
    threads of one launch: periodic data, every period bit for bit that of a short line."""
    n, periods = 100, 1343000
    kw = dict(nx=1, ny=1, dx=0.1, dy=0.1, dz=0.1, model=S.EULER, dtype=S.F32)
    small, large = S.Config(nz=n, **kw), S.Config(nz=n * periods, **kw)
    z = torch.arange(n, device="cuda", dtype=torch.float32) * (2 * np.pi / n)
    W = torch.ones(small.shape, device="cuda")
    W[0, :, 0, 0] += 0.2 * torch.sin(z)
    W[3, :, 0, 0] = 0.3 * torch.cos(z)
    U = S.prim_to_cons(small, W, S.empty_state(small))
    R = S.rhs(small, U, torch.empty_like(U))
    U = U.repeat(1, periods, 1, 1)
    got = S.rhs(large, U, torch.full_like(U, float("nan")))
    assert torch.equal(got.view(5, periods, n), R.view(5, 1, n).expand(5, periods, n))


@pytest.mark.parametrize("shape", [(16, 16, 9), (33, 17, 3), (50, 35, 7)])
@pytest.mark.parametrize("kw", [dict(model=S.DIM, thinc=1), dict(model=S.DIM, recon=1, dtype=S.F32),
                                dict(model=S.EULER, recon=1), dict(model=S.EULER, scheme=1, dtype=S.F32),
                                dict(model=S.NS, recon=1, scheme=1), dict(model=S.NS, visc_law=2, sutherland=0.4)])
def test_every_cell_is_reached_by_the_other_variants(shape, kw):
    members, alone = [], []
    for k in range(2):
        cfg = S.Config(nx=shape[0], ny=shape[1], nz=shape[2], dx=0.1, dy=0.12, dz=0.09, mu=1e-2, gamma2=1.66,
                       bc=(S.PERIODIC,) * 6 if k else (S.ZERO_GRADIENT,) * 6, **kw)
        rng = np.random.default_rng(11 + k)
        W = 1.0 + 0.1 * rng.random(cfg.shape)
        if cfg.model == S.DIM:
            W[6] = 0.2 + 0.6 * rng.random(W[6].shape)
        U = S.prim_to_cons(cfg, torch.from_numpy(W).to("cuda", cfg.torch_dtype).contiguous(), S.empty_state(cfg))
        V = U.clone()
        S.advance(cfg, V, 2, 0.0, S.workspace(cfg))
        assert torch.isfinite(V).all()
        alone.append(V)
        members.append((cfg, U, S.workspace(cfg)))
    b = S.Batch(2)
    b.set(members, fresh=[1, 1])
    b.step(2)
    torch.cuda.synchronize()
    for (_, U, _), V in zip(members, alone):
        assert torch.equal(U, V)
    b.close()
