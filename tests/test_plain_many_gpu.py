"""Plain calls over several items: large ones binned, small ones in one direct
launch, items that only push and empty ones among them.  States of the float64
form against the oracle and grids to the parity tests' 1e-12 of the absolute sum;
the launches that the call takes are counted."""

import numpy as np
import pytest

from tests import _cmp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("small,large,most", [(40, 0, 2), (40, 1, 6), (1, 0, 5), (0, 2, 9)])
def test_many_items(small, large, most):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_2602_23434_amd import binding as B
    from paper_2602_23434_amd import driver, inputs
    print(f"[plain] {small} small and {large} large items", flush=True)
    rng = np.random.default_rng(41)
    n = (8, 6, 8)
    box = inputs.Box(ndim=3, n=n, fields=inputs.turbulent_fields(n, 3, 4))
    counts = [600 + 7 * i for i in range(small)] + [60_000 + i for i in range(large)] + ([0, 3] if small > 1 else [])
    items = [inputs.Item(0, 0, inputs.make_particles(inputs.uniform_positions(rng, c, n, 3),
                                                     inputs.maxwellian_u(rng, c, 0.05))) for c in counts]
    wl = inputs.Workload("many", [box], [inputs.Species("lorentz")], items, dt=0.05, steps=2)
    ores = oracle.run_workload(wl)
    run = driver.Run(wl, prec=B.PL_F64, algo=B.PL_ALGO_PLAIN, sort_buffers=False, eng=False)
    for s in range(2):
        before = B.pl_part_stats(run.ctx)[0]
        run.step()
        launches = B.pl_part_stats(run.ctx)[0] - before
    assert run.sync() == B.PL_OK
    assert launches <= most, launches
    for i, c in enumerate(counts):
        if c == 0:
            continue
        gx, gu, gid, _ = run.state(i)
        ex, eu = _cmp.state_errors(gx, gu, gid, ores[i]["x"], ores[i]["u"], n, 3)
        assert ex <= 1e-11 and eu <= 1e-12, (i, ex, eu)
        for name, (mx, _, _) in _cmp.moment_errors(run.moments(i), ores[i]["moments"], ores[i]["abs"]).items():
            assert mx <= 1e-12, (i, name, mx)
    run.close()
