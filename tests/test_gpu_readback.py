"""dugks_phi, dugks_distributions and dugks_history at sides where a thread's
columns (two in FP32) meet the edges: odd rows, strips of 58 columns, one more
than a block's columns.  phi is the sum of the distributions in order, so the
same sum in torch agrees bitwise; the history of the first state is phi0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,flags", [(0, 0), (1, 0), (1, 2)])
@pytest.mark.parametrize("nx,ny", [(8, 8), (57, 9), (58, 8), (59, 11), (117, 10), (513, 8)])
def test_readback(precision, flags, nx, ny):
    import torch
    from paper_2007_07760_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print(f"case {nx}x{ny} prec={precision} flags={flags}", flush=True)
    rng = np.random.default_rng(nx)
    phi0 = rng.uniform(0.0, 1.0, (ny, nx))
    s = Solver(nx, ny, 0.02, 4.0, 0.5, precision=precision, vel_param=(0.02, 0.01),
               flags=flags).init(phi0)
    first = torch.as_tensor(phi0).to(device=s.device, dtype=s.dtype)
    assert torch.equal(s.history(), first)
    for _ in range(2):
        f = s.distributions()
        total = f[0].clone()
        for i in range(1, 9):
            total += f[i]
        assert torch.equal(s.phi(), total)
        s.step(1)
    # the cells are where they were put: phi moves by far less than it varies
    s.init(phi0)
    assert float((s.phi() - first).abs().max()) < 1e-5


def test_stream_is_the_current_one():
    import torch
    from paper_2007_07760_amd.batch import Batch
    from paper_2007_07760_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    side = torch.cuda.Stream()
    for ctx in (torch.cuda.stream(torch.cuda.default_stream()), torch.cuda.stream(side)):
        with ctx:
            assert Solver.stream() == Batch.stream() == torch.cuda.current_stream().cuda_stream
