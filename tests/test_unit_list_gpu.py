"""The list of work units where it takes several scans: more tiles than a scan
looks at, a number that is no multiple of a thread's tiles, more heavy tiles than
are ranked, and crowded ones among them; against the definition, exactly."""

import numpy as np
import pytest

from tests.test_runs_gpu import expected_units

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,clumps,share", [
    ((60, 52, 44), 3, 1.0),          # 2145 tiles, crowded ones cut into pieces
    ((60, 52, 96), 0, 0.35),         # 4680 tiles, about 1600 heavy ones
    ((60, 52, 96), 4, 0.35),
    ((32, 256, 8), 0, 1.0),          # 1024 tiles: half a scan
])
def test_units_of_many_tiles(n, clumps, share):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_23434_amd import binding as B
    from paper_2602_23434_amd import driver, inputs
    print(f"[units] {n} {clumps} clumps, particles in {share} of the tiles", flush=True)
    rng = np.random.default_rng(53)
    tile = (4, 4, 4)
    nt = [n[a] // tile[a] for a in range(3)]
    tiles = rng.permutation(nt[0] * nt[1] * nt[2])[:int(share * nt[0] * nt[1] * nt[2])]
    at = rng.choice(tiles, 40 * len(tiles))
    corner = np.stack([at % nt[0], at // nt[0] % nt[1], at // (nt[0] * nt[1])]) * 4.0
    x = corner + rng.random(corner.shape) * 3.999
    if clumps:
        x = np.concatenate([x, inputs.clumped_positions(rng, 90_000, clumps, 1.0, n)], axis=1)
    wl = inputs.Workload("units", [inputs.Box(ndim=3, n=n, fields=inputs.uniform_fields(n))], [inputs.Species("lorentz")],
                         [inputs.Item(0, 0, inputs.make_particles(x, np.zeros_like(x)))], dt=0.05, steps=1)
    run = driver.Run(wl, prec=B.PL_F32_OFFSET, algo=B.PL_ALGO_RUNS, tile=tile)
    run.sort()
    assert run.sync() == B.PL_OK
    npart, ntiles = x.shape[1], nt[0] * nt[1] * nt[2]
    got = run.raw(0)["runs"].astype(np.int64)
    counts = got[npart:npart + ntiles]
    want = expected_units(counts)
    units = got[npart + 3 * ntiles + 2 * B.PL_RUNS_SPLIT_UNITS]
    if share < 1.0 and not clumps:
        assert np.count_nonzero(counts > 2 * (counts.sum() // ntiles) + 1) > 1024
    if clumps:
        assert np.any(want[:, 1] >> 16 > 1)
    assert units == len(want)
    assert np.array_equal(got[npart + ntiles:npart + ntiles + 2 * units].reshape(-1, 2), want)
    run.close()
