"""Sweeps with the four sites of a block as bytes of a word (L = 8 and 16,
populations too small to fill words with replicas) against the CPU oracle: one
replica a lane and two, several sets and passes a workgroup, ragged ends, bit
rows, cluster moves.  Spins, energies, families and integer records bit for
bit, observables within 1e-12."""
import pytest

import oracle
import pamc_inputs as pi
from parity import THREADS, compare_run, compare_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,R,nT,NS,bmax,opts", [
    (8, 1, 6, 3, 4.0, {}), (8, 5, 7, 3, 5.0, dict(packed=True)), (8, 333, 9, 4, 4.0, dict(fuse_gather=False)),
    # two replicas a lane, four sets a workgroup, rows left over
    (8, 4099, 4, 2, 3.0, {}), (8, 4101, 4, 2, 3.0, dict(packed=True)),
    # tiles of several passes, the last one ragged
    (8, 61, 6, 3, 4.0, dict(tile_rows=24)), (8, 130, 6, 3, 4.0, dict(tile_rows=128)),
    (8, 40, 6, 5, 4.0, dict(icm_rounds=2)),
    (16, 1, 5, 2, 4.0, {}), (16, 7, 5, 3, 5.0, dict(packed=True)), (16, 30, 5, 3, 4.0, dict(tile_rows=6)),
    # eight waves a replica: two replicas a lane from 512 rows on
    (16, 517, 3, 1, 2.0, {}), (16, 9, 4, 4, 3.0, dict(icm_rounds=1)),
])
def test_site_words_bit_exact(L, R, nT, NS, bmax, opts):
    from paper_1710_09025_amd import Pamc

    J, beta, seed = pi.pm_j_couplings(L, 1100 + L), pi.linear_beta(bmax, nT), 1200 + R
    steps = list(range(nT))
    p = Pamc(L, J, R, beta, NS, seed, overlap_steps=steps, **opts)
    o = oracle.Oracle(L, J, R, beta, NS, seed, overlap_steps=steps, threads=THREADS,
                      **({"icm_rounds": opts["icm_rounds"]} if "icm_rounds" in opts else {}))
    what = f"L={L} R={R} {opts}"
    assert p.anneal() == o.run() == 0
    compare_run(p.observables(), p.step_sums(), o, what=what)
    compare_state(p.get_state(), o.get_state(), what)
