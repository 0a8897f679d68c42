"""The tile kernel (tile heights up to 8: one wavefront per row of a tile)
against the marching kernel (16 rows) on the same grids.  Both evaluate the
same expressions in the same order, so distributions, history and the fused
mass correction agree bitwise: no tolerance.  Sides at the edges of strips (58
columns), tiles (4 and 8 rows) and the smallest grid (8 x 8)."""
import pytest

from paper_2007_07760_amd import inputs as I

pytestmark = pytest.mark.gpu

SIDES = [(8, 8), (9, 11), (58, 12), (59, 13), (61, 17), (130, 97)]
# recon, flags, scheme, velocity kind
FORMS = [(0, 0, 0, 0), (1, 0, 0, 2), (1, 2, 0, 1), (2, 0, 0, 3), (2, 2, 0, 4), (1, 0, 0, 4),
         (3, 0, 0, 2), (3, 2, 0, 1), (1, 0, 1, 3), (1, 2, 1, 4), (0, 2, 1, 1), (2, 0, 1, 2)]
PARAMS = {0: (0.03, -0.02), 1: (0.002, 20.0, 9.0), 2: (0.05, 90.0), 3: (0.04, 70.0), 4: ()}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("recon,flags,scheme,vel", FORMS)
def test_tile_equals_march_bitwise(precision, recon, flags, scheme, vel):
    import numpy as np
    import torch
    from paper_2007_07760_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    for nx, ny in SIDES:
        print(f"case {nx}x{ny} prec={precision} recon={recon} flags={flags} scheme={scheme} "
              f"vel={vel}", flush=True)
        r = min(nx, ny)
        phi0 = I.random_circles(nx, ny, 2, 0.15 * r, 0.3 * r, 4.0, seed=nx + ny)
        uv = np.stack([0.05 * np.sin(2 * np.pi * np.arange(nx) / nx)[None, :].repeat(ny, 0),
                       0.04 * np.cos(2 * np.pi * np.arange(ny) / ny)[:, None].repeat(nx, 1)])

        def state(rows):
            return Solver(nx, ny, 0.02, 4.0, 0.5, recon=recon, precision=precision,
                          vel_kind=vel, vel_param=PARAMS[vel], flags=flags, tile_rows=rows,
                          scheme=scheme).init(phi0, uv if vel == 4 else None).step(7)

        march = state(16)
        for rows in (4, 8, 0):
            s = state(rows)
            assert torch.equal(s.distributions(), march.distributions()), (nx, ny, rows)
            assert torch.equal(s.history(), march.history()), (nx, ny, rows)
            assert s.mass() == march.mass() and s.status() == march.status()


# sides at the edges of the rule for forming the correction in the step kernel:
# 12 strips, 64 groups of 8 rows and (T2) 256 groups in all do, one more does not
@pytest.mark.parametrize("nx,ny,scheme", [(640, 168, 0), (696, 170, 0), (697, 40, 0),
                                          (58, 512, 0), (20, 513, 0), (696, 512, 1)])
def test_correction_formed_in_the_step(nx, ny, scheme):
    """Corrected plans: six steps in one call (the correction formed from the
    last step's partials by the step kernel) against six calls (each with the
    reduction kernel) and the march; bitwise, with the mass and the status.
    The blow-up of one cell is reported by all."""
    import torch
    from paper_2007_07760_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print(f"case {nx}x{ny} scheme={scheme}", flush=True)
    r = min(nx, ny)
    phi0 = I.random_circles(nx, ny, 3, 0.1 * r, 0.3 * r, 4.0, seed=nx)
    for bad in (False, True):
        if bad:
            phi0 = phi0.copy()
            phi0[ny // 2, nx // 3] = 1e38   # its square overflows in FP32

        def start(rows):
            return Solver(nx, ny, 0.02, 4.0, 0.5, precision=1, vel_kind=1,
                          vel_param=(0.0005, nx / 2, ny / 2), flags=2, tile_rows=rows,
                          scheme=scheme).init(phi0)

        one, many, march = start(8).step(6), start(8), start(16).step(6)
        for _ in range(6):
            many.step(1)
        for s in (many, march):
            assert s.status() == one.status()
            if not bad:
                assert torch.equal(s.distributions(), one.distributions())
                assert torch.equal(s.history(), one.history())
                assert s.mass() == one.mass()
        assert (one.status() != 0) == bad


# upwind-5 grids of three rounds of 8-row blocks and two of 10-row ones: the rule
# takes 10; heights that leave a last tile of 1, 5, 9 and 10 rows
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nx,ny", [(9, 4101), (59, 2055), (130, 1389), (130, 1380)])
def test_ten_row_tiles_equal_march_bitwise(precision, nx, ny):
    import torch
    from paper_2007_07760_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print(f"case {nx}x{ny} prec={precision}", flush=True)
    phi0 = I.random_circles(nx, ny, 3, 0.2 * nx, 0.4 * nx, 4.0, seed=ny)

    def state(rows):
        return Solver(nx, ny, 0.02, 4.0, 0.5, recon=3, precision=precision, vel_kind=2,
                      vel_param=(0.05, 90.0), tile_rows=rows).init(phi0).step(5)

    march = state(16)
    for rows in (8, 0):
        s = state(rows)
        assert torch.equal(s.distributions(), march.distributions()), rows
        assert torch.equal(s.history(), march.history()), rows
        assert s.mass() == march.mass() and s.status() == march.status()
