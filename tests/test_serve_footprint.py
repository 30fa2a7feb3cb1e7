"""The server's estimate of a solve's device bytes covers what the cluster
solver allocates for the solves it takes."""
import numpy as np
import pytest

import cnfgen

hm = pytest.importorskip("paper_2402_03640_amd")


def _arena(p, k, weighted, restarts):
    """Device bytes of a cluster solve next to the plan, from its layout: list
    sizes, slots, tiles, record blocks of 8 columns for 64 rows, clause entries
    by slot, best assignments, flags and exchange buffers."""
    blocks = p.v_ent_len // 64 // 8 + p.v_tiles
    words = (256 if p.n_act > 30720 else 128) + 1024 * (1 if k <= 3 else 2)
    slots = (p.v_tiles + 31) // 32 * 32 * 64
    return (blocks * (4 * words + (4096 if weighted else 0)) + 4 * p.c_ent_len + 8 * p.n_act + 4 * slots + 8 * p.v_tiles
            + restarts * (p.n + 512 * 32 + (16 if slots <= 4096 else 8) * slots + 1024))


@pytest.mark.parametrize("n,m,k", [(700, 3000, 3), (1000, 4200, 0), (4000, 17000, 3), (9000, 45000, 4), (12000, 100000, 5),
                                   (20000, 86000, 3), (28000, 120000, 0), (33000, 140000, 3), (60000, 250000, 3)])
@pytest.mark.parametrize("weighted,restarts", [(False, 1), (True, 1), (False, 9), (True, 64)])
def test_footprint_covers_a_cluster_solve(n, m, k, weighted, restarts):
    from paper_2402_03640_amd.serve import footprint_bytes
    lits = cnfgen.mixed_kcnf(n, m, seed=n) if k == 0 else cnfgen.uniform_kcnf(n, m, k, seed=n)
    p = hm._lib.Plan(n, lits)
    if p.n_heavy:
        pytest.skip("not an instance for clusters")
    L = int(np.count_nonzero(lits))
    plan = 4 * (2 * p.c_ent_len + p.v_ent_len) + 16 * (p.c_tiles + p.v_tiles) + 4 * n + (8 * 64 * p.c_tiles if weighted else 0)
    need = plan + _arena(p, 4 if k == 0 else k, weighted, restarts)
    got = footprint_bytes(n, m, L, restarts, weighted)
    assert need <= got, (need, got)
