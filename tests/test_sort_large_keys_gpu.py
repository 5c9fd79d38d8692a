"""Items whose cells add up to 2^32 in one sort call: no particle's key may be
the value that the run table's builder takes for "no neighbour".  Every array,
tile offset and run table against the same items sorted one by one, bit for bit,
with particles in the last cell of the box."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("key", [1, 3])
def test_four_items_of_the_largest_box(key):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_23434_amd import binding as B
    print(f"[sort] four items of 1024^3 cells, key {key}", flush=True)
    n, tile, count, ntiles = 1024, 8, 900, 128 ** 3
    dev = dict(device="cuda")
    bx = (B.pl_box_desc * 1)()
    for a in range(3):
        bx[0].n[a], bx[0].dx[a], bx[0].tile[a] = n, 1.0, tile
    sp = (B.pl_species_desc * 1)()
    sp[0].kind, sp[0].q, sp[0].m, sp[0].weight = B.PL_LORENTZ, 1.0, 1.0, 1.0
    d = B.pl_init_desc()
    d.ndim, d.prec, d.shape, d.algo, d.key_mode = 3, B.PL_F32_OFFSET, B.PL_TSC, B.PL_ALGO_RUNS, key
    d.c, d.nboxes, d.boxes, d.nspecies, d.species = 1.0, 1, bx, 1, sp
    d.max_items, d.max_np = 4, 4 * count
    ctx = B.pl_part_init(d)

    def make():
        """The four items and what they hold: arrays by name, each item's own."""
        items, hold = (B.pl_item * 4)(), []
        r = np.random.default_rng(17)
        for i in range(4):
            c = r.integers(0, n, (3, count))
            c[:, ::7] = n - 1                                  # the last cell of the box
            cell = (c[0] | c[1] << 10 | c[2] << 20).astype(np.uint32).view(np.int32)
            h = {"cell": [torch.tensor(cell, **dev), torch.zeros(count, dtype=torch.int32, **dev)],
                 "x": [torch.tensor(r.uniform(-0.5, 0.49, (3, count)).astype(np.float32), **dev),
                       torch.zeros((3, count), dtype=torch.float32, **dev)],
                 "u": [torch.tensor(r.normal(size=(3, count)).astype(np.float32), **dev),
                       torch.zeros((3, count), dtype=torch.float32, **dev)],
                 "id": [torch.arange(count, dtype=torch.int64, **dev), torch.zeros(count, dtype=torch.int64, **dev)],
                 "tile_start": torch.zeros(ntiles + 1, dtype=torch.int32, **dev),
                 "runs": torch.zeros(B.runs_len(count, ntiles), dtype=torch.int32, **dev)}
            p = items[i].p
            p.n, p.cur = count, 0
            for s in range(2):
                p.cell[s], p.id[s] = h["cell"][s].data_ptr(), h["id"][s].data_ptr()
                for a in range(3):
                    p.x[s][a], p.u[s][a] = h["x"][s][a].data_ptr(), h["u"][s][a].data_ptr()
            p.tile_start, p.runs = h["tile_start"].data_ptr(), h["runs"].data_ptr()
            hold.append(h)
        torch.cuda.synchronize()
        return items, hold

    together, a = make()
    B.pl_part_sort(ctx, together)
    assert B.pl_part_sync(ctx) == B.PL_OK
    single, b = make()
    for i in range(4):
        B.pl_part_sort(ctx, single[i])
    assert B.pl_part_sync(ctx) == B.PL_OK
    for i in range(4):
        for k in ("cell", "x", "u", "id"):
            assert torch.equal(a[i][k][1], b[i][k][1]), (i, k)
        assert torch.equal(a[i]["tile_start"], b[i]["tile_start"]) and torch.equal(a[i]["runs"], b[i]["runs"]), i
        # the last tile's runs: every particle of the last cell is in one
        assert int(a[i]["tile_start"][ntiles]) == count
        last = int(a[i]["runs"][count + ntiles - 1])
        beg = int(a[i]["tile_start"][ntiles - 1])
        lens = (a[i]["runs"][beg:beg + last] & 3) + 1
        assert int(lens.sum()) == count - beg >= len(range(0, count, 7))
    B.pl_part_finalize(ctx)
