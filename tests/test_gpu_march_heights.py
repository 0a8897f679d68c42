"""Tilings that the default rules and the other tests' sizes pass by: the march in
the interleaved order with uneven bands, at heights of 1 to 8 on grids too large
for the tile kernel, and uncorrected tiles of 8 rows of the tile kernel; bitwise the
same grid at 16 rows."""
import numpy as np
import pytest

from paper_2007_07760_amd import inputs as I

pytestmark = pytest.mark.gpu

PARAMS = {0: (0.03, -0.02), 2: (0.05, 90.0), 4: ()}
# nx, ny, recon, flags, scheme, velocity kind, precisions, heights
CASES = {
    # 45, 40 and 34 segments of the last height short, on 8 XCDs
    "interleaved": (150, 401, 1, 0, 0, 2, (0, 1), (9, 10, 12)),
    "interleaved corrected": (800, 905, 1, 2, 0, 2, (1,), (8, 16, 24)),
    "interleaved central-4 arrays": (75, 402, 2, 0, 0, 4, (0, 1), (9, 12)),
    # marched at the height asked for
    "short T3S3": (700, 563, 1, 0, 1, 2, (0,), (5, 8)),
    "short corrected": (1003, 903, 1, 2, 0, 0, (0, 1), (1, 8)),
    "short upwind-5": (800, 803, 3, 0, 0, 2, (1,), (7, 8)),
    # 8-row blocks: more than 256 tiles of 4 rows
    "blocks central-2": (262, 221, 0, 0, 0, 2, (0,), (8,)),
    "blocks arrays": (262, 222, 1, 0, 0, 4, (0,), (8,)),
    "blocks upwind-5": (301, 229, 3, 0, 0, 2, (0, 1), (8,)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_heights_agree_bitwise(name):
    import torch
    from paper_2007_07760_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    nx, ny, recon, flags, scheme, vel, precisions, heights = CASES[name]
    r = min(nx, ny)
    phi0 = I.random_circles(nx, ny, 3, 0.1 * r, 0.3 * r, 4.0, seed=nx)
    uv = np.stack([0.05 * np.sin(2 * np.pi * np.arange(nx) / nx)[None, :].repeat(ny, 0),
                   0.04 * np.cos(2 * np.pi * np.arange(ny) / ny)[:, None].repeat(nx, 1)])
    for precision in precisions:
        print(f"case {name} prec={precision}", flush=True)

        def state(rows):
            return Solver(nx, ny, 0.02, 4.0, 0.5, recon=recon, precision=precision,
                          vel_kind=vel, vel_param=PARAMS[vel], flags=flags, tile_rows=rows,
                          scheme=scheme).init(phi0, uv if vel == 4 else None).step(5)

        march = state(16 if 16 not in heights else 40)
        for rows in heights:
            s = state(rows)
            assert torch.equal(s.distributions(), march.distributions()), rows
            assert torch.equal(s.history(), march.history()), rows
            assert s.mass() == march.mass() and s.status() == march.status(), rows
