"""Device memory that a context takes: the sort's four words per particle, the
tables, and little more, whatever the spectral update could use."""

import pytest

pytestmark = pytest.mark.gpu


def test_context_memory():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_23434_amd import binding as B
    print("[init] memory of a context for 512^3 cells and particles", flush=True)
    n = 512
    bx = (B.pl_box_desc * 1)()
    for a in range(3):
        bx[0].n[a], bx[0].dx[a], bx[0].tile[a] = n, 1.0, 8
    sp = (B.pl_species_desc * 1)()
    sp[0].kind, sp[0].q, sp[0].m, sp[0].weight = B.PL_LORENTZ, 1.0, 1.0, 1.0
    d = B.pl_init_desc()
    d.ndim, d.prec, d.shape, d.algo, d.key_mode = 3, B.PL_F64, B.PL_TSC, B.PL_ALGO_RUNS, B.PL_KEY_TILE_RUN
    d.c, d.nboxes, d.boxes, d.nspecies, d.species = 1.0, 1, bx, 1, sp
    d.max_items, d.max_np = 4, n ** 3
    torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx = B.pl_part_init(d)
    taken = free - torch.cuda.mem_get_info()[0]
    B.pl_part_finalize(ctx)
    assert 16 * n ** 3 <= taken <= 16 * n ** 3 + (160 << 20), taken
