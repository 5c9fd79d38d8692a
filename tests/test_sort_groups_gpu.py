"""Items sorted together in one call against the same items sorted one by one:
every array, tile offset and run table bit for bit.  More items than one group
takes, an empty item, species with other arrays in between, counts on both sides
of the block sizes and of the scanned histogram."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("algo,key", [("tiled", 0), ("tiled", 1), ("tiled", 2), ("runs", 1), ("runs", 3)])
def test_group_matches_single(prec, algo, key):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_23434_amd import binding as B
    from paper_2602_23434_amd import driver, inputs
    print(f"[sort] groups {prec} {algo} {key}", flush=True)
    counts = [600_011, 1, 0, 2048, 2049, 8193, 300_007, 64, 63, 4097, 1000]
    n = (24, 16, 20)
    rng = np.random.default_rng(11)
    boxes = [inputs.Box(ndim=3, n=n, fields=inputs.uniform_fields(n)), inputs.Box(ndim=3, n=(16, 16, 16),
                                                                                  fields=inputs.uniform_fields((16, 16, 16)))]
    items = []
    for i, c in enumerate(counts):
        b = i % 2
        x = inputs.uniform_positions(rng, c, boxes[b].n, 3)
        items.append(inputs.Item(b, 0, inputs.make_particles(x, inputs.maxwellian_u(rng, c, 0.05))))
    wl = inputs.Workload("groups", boxes, [inputs.Species("lorentz")], items, dt=0.05, steps=1)
    kw = dict(prec=B.PL_F64 if prec == "f64" else B.PL_F32_OFFSET, key_mode=key,
              algo=B.PL_ALGO_TILED if algo == "tiled" else B.PL_ALGO_RUNS)
    a, b = driver.Run(wl, **kw), driver.Run(wl, **kw)
    B.pl_part_sort(a.ctx, a.items)
    for i in range(len(counts)):
        B.pl_part_sort(b.ctx, b.items[i])
    assert a.sync() == B.PL_OK and b.sync() == B.PL_OK
    assert [it.p.cur for it in a.items] == [it.p.cur for it in b.items] == [1] * len(counts)
    for i, c in enumerate(counts):
        ra, rb = a.raw(i), b.raw(i)
        for k in ra:
            va, vb = ra[k], rb[k]
            pairs = zip(va, vb) if isinstance(va, list) else [(va, vb)]
            assert all(np.array_equal(p, q) for p, q in pairs), (i, c, k)
    a.close()
    b.close()
