"""The spectral update from interleaved fluid records (one item of 32768
particles or more) against the same update from the fields (the same item beside
a second one): bit for bit, since both add the same terms in the same order."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("shape", ["tsc", "cic"])
@pytest.mark.parametrize("nb,ppc,npart", [(16, 4, 32768 + 37), (15, 1, 13440 * 4)])
def test_records_match_fields(prec, shape, nb, ppc, npart):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_23434_amd import binding as B
    from paper_2602_23434_amd import driver, inputs
    print(f"[spectra] records {prec} {shape} {nb} {npart}", flush=True)
    wl = inputs.spectra_box(n=(28, 20, 24), ppc=4, nb=nb, steps=2)
    wl.shape = shape
    p = wl.items[0].particles
    order = np.random.default_rng(7).permutation(p.n)[:npart]
    few = np.arange(50)
    wl.items = [inputs.Item(0, 0, inputs.make_particles(p.x[:, order], p.u[:, order])),
                inputs.Item(0, 0, inputs.make_particles(p.x[:, few], p.u[:, few]))]
    got = []
    for nitems in (1, 2):
        run = driver.Run(wl, prec=B.PL_F64 if prec == "f64" else B.PL_F32_OFFSET, algo=B.PL_ALGO_PLAIN,
                         spectra=True, spectra_sets=1, sort_buffers=False)
        launches = B.pl_part_stats(run.ctx)[0]
        for _ in range(wl.steps):
            B.pl_part_spectra(run.ctx, (B.pl_item * nitems)(*run.items[:nitems]), wl.dt, 1e-4, 0.5, 0.5)
        assert run.sync() == B.PL_OK
        assert B.pl_part_stats(run.ctx)[0] - launches == wl.steps * (2 if nitems == 1 else 1)
        got.append(run.spectra_state(0))
        run.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
