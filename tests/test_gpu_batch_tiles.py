"""Batches over block tiles (tile_rows = 8, and by default where the grids are
few) against the same grids over marching tiles and alone: bitwise, as every
tiling is.  Grids that stop at their own targets, graph replays after the list
changes from one kind of tile to the other, and the allocation-free step."""
import pytest

from paper_2007_07760_amd import inputs as I

pytestmark = pytest.mark.gpu

GRIDS = [(8, 8, 0, (0.03, -0.02)), (59, 13, 1, (0.002, 20.0, 9.0)), (130, 97, 2, (0.05, 90.0)),
         (58, 40, 3, (0.04, 70.0)), (200, 64, 1, (0.001, 100.0, 32.0))]
TARGETS = [3, 9, 20, 12, 16]


@pytest.fixture(scope="module")
def lib():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2007_07760_amd import _lib
    _lib.load()
    return _lib


def _solver(lib, g, precision, recon, flags, scheme):
    from paper_2007_07760_amd.solver import Solver
    nx, ny, kind, prm = g
    r = min(nx, ny)
    phi0 = I.random_circles(nx, ny, 2, 0.15 * r, 0.3 * r, 4.0, seed=nx + ny)
    return Solver(nx, ny, 0.02, 4.0, 0.5, recon=recon, precision=precision, vel_kind=kind,
                  vel_param=prm, flags=flags, scheme=scheme).init(phi0)


@pytest.mark.parametrize("precision,recon,flags,scheme", [
    (1, 1, 2, 0), (1, 1, 0, 0), (0, 1, 0, 0), (0, 2, 0, 0), (0, 0, 0, 0), (0, 1, 0, 1),
    (1, 2, 2, 1)])
def test_block_tiles_equal_marching_tiles(lib, precision, recon, flags, scheme):
    import torch
    from paper_2007_07760_amd.batch import Batch
    print(f"case prec={precision} recon={recon} flags={flags} scheme={scheme}", flush=True)
    results = []
    for rows in (8, 16, None):
        b = Batch(len(GRIDS), precision, recon, flags | (lib.BATCH_T3S3 if scheme else 0))
        sol = [_solver(lib, g, precision, recon, flags, scheme) for g in GRIDS]
        for k, s in enumerate(sol):
            b.set(k, s, TARGETS[k])
        if rows:
            b.tile_rows = rows
        b.commit()
        b.step(8, graph_steps=4)
        if rows:                       # the other kind of tile, the graph of the first kept
            b.tile_rows = 24 - rows
            b.commit()
        b.step(8, graph_steps=4)
        if rows:
            b.tile_rows = rows
            b.commit()
        b.step(8, graph_steps=4)
        b.sync()
        assert [s.step_index for s in sol] == TARGETS
        results.append([(s.distributions(), s.history(), s.mass()) for s in sol])
    for k, g in enumerate(GRIDS):
        s = _solver(lib, g, precision, recon, flags, scheme).step(TARGETS[k])
        alone = (s.distributions(), s.history(), s.mass())
        for r in results:
            assert torch.equal(r[k][0], alone[0]) and torch.equal(r[k][1], alone[1]), g
            assert r[k][2] == alone[2], g


@pytest.mark.parametrize("precision,recon,flags,scheme", [(1, 2, 2, 0), (0, 0, 0, 0), (0, 2, 0, 1)])
def test_allocation_free_step_over_block_tiles(lib, precision, recon, flags, scheme):
    import torch
    print(f"case noalloc prec={precision} recon={recon} flags={flags} scheme={scheme}", flush=True)
    many, alone = ([_solver(lib, g, precision, recon, flags, scheme) for g in GRIDS]
                   for _ in range(2))
    lib.dugks_step_many_noalloc([s.plan for s in many], [s.state.data_ptr() for s in many],
                                [0] * len(many), 9, torch.cuda.current_stream().cuda_stream)
    for s, o, g in zip(many, alone, GRIDS):
        s.step_index = 9
        o.step(9)
        assert torch.equal(s.distributions(), o.distributions()), g
        assert torch.equal(s.history(), o.history()) and s.mass() == o.mass(), g
