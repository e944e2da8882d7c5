"""Sweeps with replicas as bits of a word against the CPU oracle, at the edges
of their shapes: words of 1 to 32 replicas, full and partial sets, passes that
end inside a word, site blocks that leave lanes idle, the largest lattices
each table of site thresholds or bond sums fits, and populations around the
sizes where the statistics change their ways.  Spins, energies, families and
integer records bit for bit, observables within 1e-12 (the oracle's
arithmetic is the same up to the order of a few sums)."""
import numpy as np
import pytest

import oracle
import pamc_inputs as pi
from parity import THREADS, compare_run, compare_state

pytestmark = pytest.mark.gpu

# (couplings, dim, L, R, n_temps, sweeps, beta_max, options)
CASES = [
    # +-1: one replica a word, a word and one replica more, several sets, lanes
    # beyond the last block (three colours), blocks in turn (L > 26), bit rows
    ("pm", 3, 6, 37, 7, 3, 4.0, dict(tile_rows=1, group_replicas=16)),
    ("pm", 3, 8, 33, 9, 3, 6.0, dict(tile_rows=32)),
    ("pm", 3, 10, 97, 7, 3, 6.0, dict(tile_rows=96, group_replicas=32)),
    ("pm", 3, 7, 130, 9, 3, 3.0, dict(tile_rows=63, group_replicas=32, packed=True)),
    ("pm", 3, 23, 5, 3, 2, 3.0, {}),
    ("pm", 3, 28, 3, 3, 2, 3.0, dict(packed=True)),
    # (a population buffer that holds less than one exported row)
    ("pm", 3, 28, 3, 3, 2, 0.01, dict(packed=True, capacity=6)),
    ("pm", 3, 4, 31300, 3, 1, 1.0, dict(capacity=32768)),
    ("pm", 3, 4, 31300, 3, 1, 1.0, dict(capacity=32769)),
    # +-1, few replicas: bytes of a word, two and three colours, one set a
    # workgroup and several, bit rows with a ragged last word
    ("pm", 3, 5, 50, 7, 3, 4.0, dict(tile_rows=3, group_replicas=16, packed=True)),
    ("pm", 3, 11, 9, 5, 3, 4.0, dict(packed=True)),
    ("pm", 3, 13, 9, 4, 2, 3.0, {}),
    ("pm", 3, 16, 31, 4, 2, 3.0, dict(tile_rows=2)),
    # the largest population whose map the statistics write, and the next
    ("pm", 3, 4, 3600, 3, 1, 1.0, dict(capacity=4096)),
    ("pm", 3, 4, 3600, 3, 1, 1.0, dict(capacity=4097)),
    ("real", 3, 4, 3600, 3, 1, 1.0, dict(capacity=4096)),
    # real: few and many replicas a word, bond sums and thresholds, at the last
    # lattice of either and the first beyond
    ("real", 3, 8, 15, 6, 3, 20.0, dict(tile_rows=4, group_replicas=4)),
    ("real", 3, 8, 401, 6, 3, 20.0, dict(tile_rows=100, group_replicas=64)),
    ("real", 3, 9, 70, 5, 2, 6.0, dict(packed=True)),
    ("real", 3, 13, 40, 4, 2, 6.0, {}),
    ("real", 3, 12, 40, 4, 2, 6.0, {}),
    ("real", 3, 14, 9, 4, 2, 6.0, {}),
    ("real", 3, 16, 70, 4, 2, 20.0, dict(tile_rows=32, group_replicas=8, packed=True)),
    ("real", 3, 20, 5, 3, 2, 6.0, {}),
    ("real", 3, 21, 4, 3, 2, 6.0, {}),
    ("real", 2, 5, 500, 8, 3, 20.0, dict(tile_rows=6, group_replicas=64)),
    ("real", 2, 45, 60, 4, 2, 6.0, {}),
    ("real", 2, 46, 60, 4, 2, 6.0, {}),
    ("real", 2, 48, 60, 4, 2, 6.0, {}),
    ("real", 2, 49, 60, 4, 2, 6.0, {}),
    ("real", 2, 64, 33, 4, 2, 6.0, dict(tile_rows=8, group_replicas=8)),
]


@pytest.mark.parametrize("model,dim,L,R,nT,NS,bmax,opts", CASES)
def test_words_bit_exact(model, dim, L, R, nT, NS, bmax, opts):
    from paper_1710_09025_amd import Pamc

    J = pi.pm_j_couplings(L, 700 + L) if model == "pm" else pi.gaussian_couplings(L, 700 + L, dim=dim)
    beta, seed = pi.linear_beta(bmax, nT), 800 + L
    opts = dict(opts)
    capacity = opts.pop("capacity", R + 8 * int(np.ceil(np.sqrt(R))) + 64)
    p = Pamc(L, J, R, beta, NS, seed, capacity=capacity, **opts)
    o = oracle.Oracle(L, J, R, beta, NS, seed, capacity=capacity, threads=THREADS)
    what = f"{model} {dim}D L={L} R={R}"
    assert p.anneal() == o.run() == 0
    compare_run(p.observables(), p.step_sums(), o, what=what)
    final = p.get_state()
    compare_state(final, o.get_state(), what)
    # a state taken back into the finished run goes on as in a new one
    half = oracle.Oracle(L, J, R, beta, NS, seed, capacity=capacity, threads=THREADS)
    half.run(nT // 2)
    s = half.get_state()
    p.set_state(s["step"], s["spins"], s["family"], s["lnZ"])
    assert p.anneal() == 0
    compare_state(p.get_state(), final, what + " after set_state")
