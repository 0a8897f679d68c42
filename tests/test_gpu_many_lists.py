"""dugks_step_many_noalloc on lists whose work list is of marching tiles (more
16-row tiles than the block tiles' limit) and on single grids: the grids'
results are bitwise those of the same grids stepped alone, whatever pieces of
them each XCD takes.  Tile heights of the plans' own, short last segments, two
calls in a row."""
import pytest

from paper_2007_07760_amd import inputs as I

pytestmark = pytest.mark.gpu

LISTS = {
    "one": [(1003, 777, 0)],                                  # block tiles, up to FP64's limit
    "one, marched": [(1500, 1283, 0)],
    "heights": [(610, 525, 24), (700, 333, 0), (8, 8, 0), (523, 771, 40), (59, 300, 16),
                (640, 640, 4), (130, 97, 64)],
    "uneven": [(1171, 1001, 32)] + [(9 + 7 * k, 11 + 5 * k, 0) for k in range(20)],
}


@pytest.mark.parametrize("precision,flags,scheme", [(1, 2, 0), (1, 0, 0), (0, 0, 0), (0, 0, 1),
                                                    (1, 2, 1)])
@pytest.mark.parametrize("name", sorted(LISTS))
def test_many_equals_alone_bitwise(name, precision, flags, scheme):
    import torch
    from paper_2007_07760_amd import _lib as C
    from paper_2007_07760_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print(f"case {name} prec={precision} flags={flags} scheme={scheme}", flush=True)

    def make():
        return [Solver(nx, ny, 0.02, 4.0, 0.5, precision=precision, vel_kind=2,
                       vel_param=(0.05, 90.0), flags=flags, scheme=scheme, tile_rows=rows)
                .init(I.random_circles(nx, ny, 3, 0.1 * min(nx, ny), 0.3 * min(nx, ny), 4.0,
                                       seed=nx + k))
                for k, (nx, ny, rows) in enumerate(LISTS[name])]

    many, alone = make(), make()
    stream = torch.cuda.current_stream().cuda_stream
    for nsteps in (3, 4):
        C.dugks_step_many_noalloc([s.plan for s in many], [s.state.data_ptr() for s in many],
                                  [s.step_index for s in many], nsteps, stream)
        for s in many:
            s.step_index += nsteps
    for s, o, g in zip(many, alone, LISTS[name]):
        o.step(7)
        assert torch.equal(s.distributions(), o.distributions()), g
        assert torch.equal(s.history(), o.history()), g
        assert s.mass() == o.mass() and s.status() == o.status() == C.OK, g


@pytest.mark.parametrize("precision,flags,scheme", [(1, 2, 0), (0, 0, 0), (0, 0, 1)])
def test_batch_of_many_rounds_with_its_own_targets(precision, flags, scheme):
    """A batch of more than two rounds of marching tiles (3072 and 2048 wavefronts)
    whose grids stop at different steps: bitwise the grids alone."""
    import torch
    from paper_2007_07760_amd import _lib as C
    from paper_2007_07760_amd.batch import Batch
    from paper_2007_07760_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print(f"case batch prec={precision} flags={flags} scheme={scheme}", flush=True)
    n = 40
    sizes = [(291 + 9 * (k % 8), 410 + k) for k in range(n)]
    targets = [1 + 5 * (k % 3) for k in range(n)]

    def make():
        return [Solver(nx, ny, 0.02, 4.0, 0.5, precision=precision, vel_kind=3,
                       vel_param=(0.04, 70.0), flags=flags, scheme=scheme)
                .init(I.random_circles(nx, ny, 3, 20.0, 60.0, 4.0, seed=k))
                for k, (nx, ny) in enumerate(sizes)]

    batched, alone = make(), make()
    b = Batch(n, precision, C.UPWIND3, flags | (C.BATCH_T3S3 if scheme else 0))
    for k, s in enumerate(batched):
        b.set(k, s, targets[k])
    b.commit()
    b.step(13, graph_steps=4)
    b.sync()
    for k, (s, o) in enumerate(zip(batched, alone)):
        o.step(targets[k])
        assert s.step_index == targets[k]
        assert torch.equal(s.distributions(), o.distributions()), k
        assert torch.equal(s.history(), o.history()) and s.mass() == o.mass(), k
