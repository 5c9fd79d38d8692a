"""The self-grouping tile kernels (binned plain calls, the tiled algorithm,
split push and deposit calls) against the oracle and the run-based kernel, at
boxes their tiles do not divide, ragged counts, crowded cells (runs beyond the
counted rounds), and fast particles (queues that overflow).

Tolerances: float64 as in the parity tests (1e-11 cells, 1e-12 max(|u|,
0.05), 1e-12 A_c).  Float32 states are the run-based kernel's bit for bit; its
deposits differ by that kernel's float32 sums of at most four terms (four
roundings, each at most 2^-24 of the batch's sum of |mu| W): 4 * 2^-24 A_c,
taken as 5 for the float32 rounding of mu inside A_c.
"""

import numpy as np
import pytest

from tests import _cmp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mods():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_2602_23434_amd import binding, driver, inputs
    binding.lib()
    return oracle, driver, inputs, binding


def _workload(inputs, name):
    if name == "2d":
        return inputs.turbulent_2d(n=(45, 70), npart=20011, steps=2)
    if name == "crowded":
        # every particle in a few cells of two tiles: hundreds per cell
        wl = inputs.turbulent_box(n=16, npart=20011, steps=2)
        x = wl.items[0].particles.x
        x[:] = np.array([[3.0], [7.0], [5.0]]) + np.mod(x, 2.0)
        return wl
    if name == "fast":
        wl = inputs.turbulent_box(n=16, npart=30011, steps=2, sigma_v=0.1)     # |v| < c for every draw
        wl.dt = 0.9
        return wl
    wl = inputs.turbulent_box(n=(37, 21, 19), npart=30011, steps=2)
    if name == "cic":
        wl.shape = "cic"
    if name == "dust":
        wl.species[0].kind, wl.species[0].t_stop = "dust", 0.1
    return wl


def _check_f64(run, ores, wl):
    gx, gu, gid, st = run.state(0)
    ex, eu = _cmp.state_errors(gx, gu, gid, ores["x"], ores["u"], wl.boxes[0].n, wl.boxes[0].ndim)
    assert ex <= 1e-11 and eu <= 1e-12, (ex, eu)
    for name, (mx, _, _) in _cmp.moment_errors(run.moments(0), ores["moments"], ores["abs"]).items():
        assert name == "eng" or mx <= 1e-12, (name, mx)


@pytest.mark.parametrize("name", ["3d", "2d", "crowded", "fast", "cic", "dust"])
@pytest.mark.parametrize("algo", ["plain", "tiled"])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_fused(mods, prec, algo, name):
    oracle, driver, inputs, B = mods
    print(f"[local] fused {prec} {algo} {name}", flush=True)
    wl = _workload(inputs, name)
    p = B.PL_F64 if prec == "f64" else B.PL_F32_OFFSET
    n = wl.boxes[0].n
    # tiles of more than 512 particles on average, so that the tiled algorithm groups them
    tile = None if algo == "plain" else tuple(next(t for t in (8, 7, 19, 5, 1) if v % t == 0) for v in n)
    if name == "3d" and algo == "tiled":
        tile = (37, 7, 1)
    ores = oracle.run_workload(wl)[0]
    run = driver.Run(wl, prec=p, algo=B.PL_ALGO_PLAIN if algo == "plain" else B.PL_ALGO_TILED, tile=tile)
    if algo == "tiled":
        run.sort()
    for _ in range(wl.steps):
        run.step()
    assert run.sync() == B.PL_OK
    if prec == "f64":
        _check_f64(run, ores, wl)
        run.close()
        return
    ref = driver.Run(wl, prec=p, algo=B.PL_ALGO_RUNS)
    ref.sort()
    for _ in range(wl.steps):
        ref.step()
    assert ref.sync() == B.PL_OK
    gx, gu, gid, _ = run.state(0)
    rx, ru, rid, _ = ref.state(0)
    assert np.array_equal(_cmp.by_id(gx, gid), _cmp.by_id(rx, rid))
    assert np.array_equal(_cmp.by_id(gu, gid), _cmp.by_id(ru, rid))
    for ch, mx in _cmp.moment_errors(run.moments(0), ref.moments(0), ores["abs"]).items():
        assert mx[0] <= 5 * 2.0 ** -24, (ch, mx)
    run.close()
    ref.close()


@pytest.mark.parametrize("name", ["3d", "crowded", "fast", "dust"])
@pytest.mark.parametrize("algo", ["plain", "tiled", "runs"])
def test_split_calls_f64(mods, algo, name):
    """A push and a deposit call give the fused step's states and grids (the
    plain calls bin their particles for each), also after the particles have
    moved since the sort."""
    oracle, driver, inputs, B = mods
    print(f"[local] split {algo} {name}", flush=True)
    wl = _workload(inputs, name)
    ores = oracle.run_workload(wl)[0]
    a = {"plain": B.PL_ALGO_PLAIN, "tiled": B.PL_ALGO_TILED, "runs": B.PL_ALGO_RUNS}[algo]
    run = driver.Run(wl, prec=B.PL_F64, algo=a, fp=True, eng=False)
    if algo != "plain":
        run.sort()
    for _ in range(wl.steps):
        run.step(flags=0)
        run.deposit()
    assert run.sync() == B.PL_OK
    _check_f64(run, ores, wl)
    run.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("rk", [2, 3])
def test_binned_tracers_match_tiled(mods, prec, rk):
    """70001 tracers in no order (binned push) and sorted into tiles: the same
    states bit for bit."""
    oracle, driver, inputs, B = mods
    wl = inputs.turbulent_box(n=(20, 24, 28), npart=70001, steps=2)
    wl.species[0].kind, wl.species[0].rk_stages = "tracer", rk
    p = B.PL_F64 if prec == "f64" else B.PL_F32_OFFSET
    got = []
    for a in (B.PL_ALGO_PLAIN, B.PL_ALGO_TILED):
        run = driver.Run(wl, prec=p, algo=a)
        if a == B.PL_ALGO_TILED:
            run.sort()
        for _ in range(wl.steps):
            run.step()
        assert run.sync() == B.PL_OK
        x, u, ids, _ = run.state(0)
        got.append((_cmp.by_id(x, ids), _cmp.by_id(u, ids)))
        run.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
