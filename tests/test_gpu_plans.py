"""GPU parity where the launch plans change their split: rounds of workgroups, shares and tables at their limits.

Each case sits at the edge of a planning rule (one workgroup count to the next, a share above the size that
earlier tables held, a remainder in the last round) and is compared with the fp64 oracle at the tolerances of
the operation's own tests.
"""
import numpy as np
import pytest

from mv_check import _rand_bits, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,Hkv,G,C,L,ld,seqs", [
    (3, 8, 1, 40, 1500, 300, [0, 2]),       # 24 units: 10 workgroups each, one round of 240
    (8, 8, 4, 256, 2500, 800, [7]),         # 256 units, one workgroup each: shares above 2,048 entries
    (9, 8, 4, 256, 2200, 700, [8]),         # 288 units: two workgroups each, three rounds
])
def test_block_workgroup_rounds(S, Hkv, G, C, L, ld, seqs):
    lens = [L] * (S - 1) + [L - 37]
    k, v = _rand_bits((S, Hkv, L, 128), 300), _rand_bits((S, Hkv, L, 128), 301)
    qb = _rand_bits((S, C, Hkv * G, 128), 302)
    g = np.random.default_rng(303)
    idx_v = np.full((1, S, Hkv, ld), -1, np.int32)
    for s in range(S):
        for h in range(Hkv):
            idx_v[0, s, h] = np.sort(g.choice(lens[s], ld, replace=False))
    _run(k, v, qb, idx_v, np.full((1, S), ld, np.int32), lens, f"rounds S={S}", seqs=seqs, seed=7)
