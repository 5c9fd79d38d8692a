"""Launches of the run kernel with more units than blocks and crowded pieces among
them, of one item and of several with other boxes: a block claims nothing beyond
a crowded piece until it is through, and goes on to light and crowded ones of any
item.  Per-id states bit-identical to the tiled algorithm's; grids to the rounding
of their sums (float64 1e-12 of the absolute sum, float32 sums of a batch 2e-6 of
the largest value, as in the other tests of split tiles)."""

import numpy as np
import pytest

from tests import _cmp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("boxes,tile", [
    ([(64, 64, 40)], (8, 8, 8)),                       # fixed shapes (float32) and run-time ones
    ([(64, 64, 32)], (8, 8, 4)),
    ([(32, 32, 32), (16, 32, 48), (32, 16, 16)], (4, 4, 4)),
])
def test_crowded_pieces_among_light_units(prec, boxes, tile):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_23434_amd import binding as B
    from paper_2602_23434_amd import driver, inputs
    print(f"[runs] heavy units {prec} {boxes} {tile}", flush=True)
    rng = np.random.default_rng(31)
    bx, items = [], []
    for b, n in enumerate(boxes):
        xc = inputs.clumped_positions(rng, 90_000 // len(boxes), 3, 1.2, n)
        xu = inputs.uniform_positions(rng, 240_000 // len(boxes), n, 3)
        x = np.concatenate([xc, xu], axis=1)
        bx.append(inputs.Box(ndim=3, n=n, fields=inputs.turbulent_fields(n, 5 + b, 9 + b)))
        items.append(inputs.Item(b, 0, inputs.make_particles(x, inputs.maxwellian_u(rng, x.shape[1], 0.05))))
    wl = inputs.Workload("heavy", bx, [inputs.Species("lorentz")], items, dt=0.05, steps=4)
    p = B.PL_F64 if prec == "f64" else B.PL_F32_OFFSET
    res = []
    for algo, key in ((B.PL_ALGO_TILED, B.PL_KEY_TILE_CELL), (B.PL_ALGO_RUNS, B.PL_KEY_TILE_RUN)):
        run = driver.Run(wl, prec=p, algo=algo, key_mode=key, tile=tile, eng=False)
        for s in range(4):
            if s % 2 == 0:
                run.sort()
            run.step()
        assert run.sync() == B.PL_OK
        if algo == B.PL_ALGO_RUNS:
            assert B.pl_part_stats(run.ctx)[4:6] == [4, 0]
            for i, n in enumerate(boxes):
                npart, nt = items[i].particles.n, int(np.prod(np.array(n) // np.array(tile)))
                units = int(run.raw(i)["runs"][npart + nt + 2 * (nt + B.PL_RUNS_SPLIT_UNITS)])
                assert units > 256 or len(boxes) > 1
        states = []
        for i in range(len(boxes)):
            raw = run.raw(i)
            ids = raw["id"].astype(np.int64)
            states.append({k: _cmp.by_id(np.stack(v) if isinstance(v, list) else v, ids) for k, v in raw.items()
                           if k in ("x", "u", "cell")})
        res.append((states, [run.moments(i) for i in range(len(boxes))]))
        run.close()
    (sa, ma), (sb, mb) = res
    for i in range(len(boxes)):
        for k in sa[i]:
            assert np.array_equal(sa[i][k], sb[i][k]), (i, k)
        for k in ma[i]:
            va, vb = np.asarray(ma[i][k]), np.asarray(mb[i][k])
            tol = 1e-12 if prec == "f64" else 2e-6
            assert np.abs(va - vb).max() <= tol * np.abs(va).max(), (i, k)
