"""Calls whose item table goes to the GPU as kernel arguments (up to four items,
the moments zeroed by the same kernel) and through the pinned ring (more),
eager calls back to back over different items, with and without zeroing, on
boxes with fewer and with more work units than blocks.  States against the oracle
with the float64 parity tests' tolerances.  Moments against recorded graphs,
whose table is copied before the recording, with those tests' 1e-12 A_c: there
the particles are the same bits, which the oracle's are not, and in the sparse
box a cell that only a weight's tail reaches multiplies that last bit."""

import numpy as np
import pytest

from tests import _cmp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("algo", ["plain", "tiled", "runs"])
@pytest.mark.parametrize("count", [1, 2, 4, 5])
def test_item_table(count, algo):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_2602_23434_amd import binding as B
    from paper_2602_23434_amd import driver, inputs
    print(f"[table] {algo} {count}", flush=True)
    sizes = [((16, 16, 16), 6007), ((8, 8, 8), 65), ((40, 24, 16), 20011), ((16, 8, 24), 1), ((64, 64, 32), 30011)]
    kinds = ["lorentz", "dust", "lorentz", "tracer", "lorentz"]
    boxes, items = [], []
    rng = np.random.default_rng(23)
    for b in range(count):
        n, c = sizes[b]
        boxes.append(inputs.Box(ndim=3, n=n, fields=inputs.uniform_fields(n)))
        items.append(inputs.Item(b, ["lorentz", "dust", "tracer"].index(kinds[b]),
                                 inputs.make_particles(inputs.uniform_positions(rng, c, n, 3),
                                                       inputs.maxwellian_u(rng, c, 0.05))))
    wl = inputs.Workload("table", boxes, [inputs.Species("lorentz"), inputs.Species("dust", t_stop=0.1),
                                          inputs.Species("tracer")], items, dt=0.05, steps=3)
    ores = oracle.run_workload(wl)
    kw = dict(prec=B.PL_F64, algo={"plain": B.PL_ALGO_PLAIN, "tiled": B.PL_ALGO_TILED,
                             "runs": B.PL_ALGO_RUNS}[algo], tile=(8, 8, 4), fp=True, eng=False)
    run, ref = driver.Run(wl, **kw), driver.Run(wl, **kw)
    for m in run.mom_blocks:
        m.fill_(7.0)
    torch.cuda.synchronize()
    if algo != "plain":
        run.sort()
        ref.sort()
    # the whole call, then item by item, then the whole call again
    run.step()
    for i in range(count):
        B.pl_part_gather_push(run.ctx, run.items[i], wl.dt, B.PL_FUSE_DEPOSIT | B.PL_ZERO_FIRST)
    run.step()
    for _ in range(3):
        ref.step(flags=B.PL_FUSE_DEPOSIT | B.PL_ZERO_FIRST | B.PL_GRAPH)
    assert run.sync() == B.PL_OK and ref.sync() == B.PL_OK
    for i in range(count):
        gx, gu, gid, _ = run.state(i)
        ex, eu = _cmp.state_errors(gx, gu, gid, ores[i]["x"], ores[i]["u"], boxes[i].n, 3)
        assert ex <= 1e-11 and eu <= 1e-12, (i, ex, eu)
        ra, rb = run.raw(i), ref.raw(i)
        for k in ("x", "u"):
            assert all(np.array_equal(p, q) for p, q in zip(ra[k], rb[k])), (i, k)
        if kinds[i] != "tracer":
            for name, (mx, _, _) in _cmp.moment_errors(run.moments(i), ref.moments(i), ores[i]["abs"]).items():
                assert mx <= 1e-12, (i, name, mx)
    # no zeroing: the same deposit again on top
    B.pl_part_deposit(run.ctx, run.items, 0)
    assert run.sync() == B.PL_OK
    for i in range(count):
        if kinds[i] == "tracer":
            continue
        twice = run.moments(i)
        assert np.allclose(np.asarray(twice["rho"]), 2 * np.asarray(ores[i]["moments"]["rho"]), rtol=0,
                           atol=2e-12 * np.abs(ores[i]["abs"]["rho"]).max()), i
    run.close()
    ref.close()
