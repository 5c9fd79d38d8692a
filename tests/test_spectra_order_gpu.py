"""The spectral update of one item of 32768 particles or more in some order of
place, which samples the fields although there is scratch for records, and in
part of one: bit for bit the update of the same item beside a second one, which
always samples the fields (both ways add the same terms in the same order)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("ndim,order", [(3, "cell"), (3, "tile"), (3, "half"), (3, "seam"), (2, "cell"), (2, "none")])
def test_orders_match_fields(prec, ndim, order):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_23434_amd import binding as B
    from paper_2602_23434_amd import driver, inputs
    print(f"[spectra] order {prec} {ndim} {order}", flush=True)
    wl = inputs.spectra_box(n=(28, 20, 24) if ndim == 3 else (120, 112, 8), ppc=4, nb=16, steps=2)
    p = wl.items[0].particles
    if ndim == 2:                                              # one plane of the box and its particles
        f = {k: np.ascontiguousarray(v[..., :1, :, :]) for k, v in wl.boxes[0].fields.items()}
        wl.boxes = [inputs.Box(ndim=2, n=(120, 112, 1), fields=f)]
        flat = p.x[2] < 1.0
        p = inputs.make_particles(p.x[:, flat], p.u[:, flat])
    rng = np.random.default_rng(7)
    at = np.arange(p.n)
    c = np.floor(p.x).astype(np.int64)
    if order == "tile":
        t = c[0] // 4 + 100 * (c[1] // 4) + 10000 * (c[2] // 4)
        at = np.lexsort((rng.random(p.n), t))
    elif order == "half":
        at = np.concatenate([at[:p.n // 2], rng.permutation(at[p.n // 2:])])
    elif order == "seam":
        at = np.lexsort((c[0] % 2, c[1], c[2]))                # pairs at both ends of a row
    elif order == "none":
        at = rng.permutation(at)
    few = np.arange(50)
    wl.items = [inputs.Item(0, 0, inputs.make_particles(p.x[:, at], p.u[:, at])),
                inputs.Item(0, 0, inputs.make_particles(p.x[:, few], p.u[:, few]))]
    got = []
    for nitems in (1, 2):
        run = driver.Run(wl, prec=B.PL_F64 if prec == "f64" else B.PL_F32_OFFSET, algo=B.PL_ALGO_PLAIN,
                         spectra=True, spectra_sets=1, sort_buffers=False)
        for _ in range(wl.steps):
            B.pl_part_spectra(run.ctx, (B.pl_item * nitems)(*run.items[:nitems]), wl.dt, 1e-4, 0.5, 0.5)
        assert run.sync() == B.PL_OK
        got.append(run.spectra_state(0))
        run.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
