"""Float32 steps of tiles whose footprint leaves them to the float64 sums: the
run-based algorithm does not take its run kernel there, and its grids agree with
the tiled algorithm's to the rounding of float64 sums (float32 sums of a batch
differ by 1e-8).  A cell adds at most a few hundred products, each rounded once:
1e-13 of the absolute sum, tested with the parity tests' 1e-12."""

import numpy as np
import pytest

from tests import _cmp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,n,eng,kernel", [
    ((16, 8, 4), (32, 16, 16), True, False),
    ((12, 8, 6), (24, 16, 18), True, False),
    ((9, 9, 8), (27, 18, 16), False, False),
    ((16, 8, 4), (32, 16, 16), False, True),
])
def test_tiles_left_to_float64_sums(tile, n, eng, kernel):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_2602_23434_amd import binding as B
    from paper_2602_23434_amd import driver, inputs
    print(f"[runs] float64 sums {tile} {eng}", flush=True)
    count = 12 * int(np.prod(n)) + 5
    rng = np.random.default_rng(29)
    wl = inputs.Workload("sums", [inputs.Box(ndim=3, n=n, fields=inputs.uniform_fields(n, E=(0.02, -0.01, 0.03)))],
                         [inputs.Species("lorentz")],
                         [inputs.Item(0, 0, inputs.make_particles(inputs.uniform_positions(rng, count, n, 3),
                                                                  inputs.maxwellian_u(rng, count, 0.05)))],
                         dt=0.05, steps=1)
    ores = oracle.run_workload(wl)
    got = []
    for algo, key in ((B.PL_ALGO_RUNS, B.PL_KEY_TILE_RUN), (B.PL_ALGO_TILED, B.PL_KEY_TILE_CELL)):
        run = driver.Run(wl, prec=B.PL_F32_OFFSET, algo=algo, key_mode=key, tile=tile, eng=eng)
        run.sort()
        run.step()
        assert run.sync() == B.PL_OK
        if algo == B.PL_ALGO_RUNS:
            stats = B.pl_part_stats(run.ctx)
            assert (stats[4], stats[5]) == ((1, 0) if kernel else (0, 1))
        got.append(run.moments(0))
        run.close()
    worst = max(mx for mx, _, _ in _cmp.moment_errors(got[0], got[1], ores[0]["abs"]).values())
    assert (worst <= 1e-12) == (not kernel), worst
