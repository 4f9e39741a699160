"""GPU parity where the launch plans change their split: rounds of workgroups, and shares that fill the slot tables.

Each case sits at the edge of a planning rule (one workgroup count to the next, a share above the size that
earlier tables held, a remainder in the last round) and is compared with the fp64 oracle at the tolerances of
the operation's own tests.
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2606_00144_amd as bd
import synth
from gpu_utils import assert_close, bf16_dev, bf16_host64, case, check_selection, i32_dev, oracle_scores, paged_kv
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


def _select_inputs(lens, Hkv, W, G, seed):
    """Keys whose norm grows with the position, so that a row's reference is raised again and again."""
    g = np.random.default_rng(seed)
    q = synth.f32_to_bf16_bits(g.standard_normal((len(lens), W, Hkv * G, 128)).astype(np.float32))
    ks = [synth.f32_to_bf16_bits((g.standard_normal((Hkv, n, 128)) * (0.2 + 5.0 * np.arange(n)[None, :, None] / n)
                                  ).astype(np.float32)) for n in lens]
    return q, ks


def _select_case(q, ks, lens, Hkv, W, G, B, layout):
    Hq, L = Hkv * G, max(lens)
    table = None
    if layout.startswith("page"):
        P = int(layout[4:])
        npg = [(n + P - 1) // P for n in lens]
        perm = np.random.default_rng(5).permutation(sum(npg) + 3)
        t, at = np.full((len(lens), max(npg)), -1, np.int32), 0
        for s, n in enumerate(npg):
            t[s, :n] = perm[at:at + n]
            at += n
        kd, _ = paged_kv(ks, ks, t, sum(npg) + 3, P)
        table = i32_dev(t)
    else:
        k = np.zeros((len(lens), Hkv, L, 128), np.uint16)
        for s, n in enumerate(lens):
            k[s, :, :n] = ks[s]
        kd = bf16_dev(k)
        if layout == "token-major":             # rows of one head Hkv * 128 elements apart
            kd = kd.transpose(1, 2).contiguous().transpose(1, 2)
    case(f"select rows={W * G} {layout} S={len(lens)}")
    idx, nsel, sc = bd.bd_select_kv(kd, bf16_dev(q), i32_dev(lens), B, return_scores=True, page_table=table, max_seq_len=L)
    torch.cuda.synchronize()
    raws = oracle_scores(ks, q, lens, Hq)
    check_selection(idx.cpu().numpy(), nsel.cpu().numpy(), sc.cpu().numpy(), raws, lens, W, B,
                    f"rows {W * G} {layout}", Hq=Hq)


@pytest.mark.parametrize("layout", ["contiguous", "token-major", "page16", "page24", "page64"])
@pytest.mark.parametrize("W,G", [(1, 1), (33, 1), (13, 5), (31, 4), (35, 5), (86, 3)])
def test_select_row_tiles(W, G, layout):
    # 1..4 row tiles of 32, one and several row blocks, a remainder in each; splits and tiles cut short
    lens = [1033, 700, 289]
    q, ks = _select_inputs(lens, 2, W, G, 41)
    _select_case(q, ks, lens, 2, W, G, 128, layout)


@pytest.mark.parametrize("S,Hkv", [(36, 4), (65, 4), (3, 2)])
def test_select_split_rounds(S, Hkv):
    # 144 units (several splits each, whole rounds), 260 (one more than a round), 6 (every key block a split)
    lens = [520 + 7 * (s % 5) for s in range(S)]
    q, ks = _select_inputs(lens, Hkv, 8, 4, 43)
    _select_case(q, ks, lens, Hkv, 8, 4, 96, "contiguous")


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("S,Hkv", [(64, 5), (9, 32), (65, 4), (2, 160)])
def test_verify_longest_first(S, Hkv, paged):
    # more whole units than CUs, caches too short for the longest-first order (test_verify_longest_first_rule has
    # both sides of that line); equal lengths, the shortest possible and the longest among them
    gamma, Lmax, Hq = 2, 150, Hkv
    g = np.random.default_rng(47)
    lens = [int(n) for n in g.choice([gamma + 1, 40, 97, 98, 150], S)]
    k, v = _rand_bits((S, Hkv, Lmax, 128), 48), _rand_bits((S, Hkv, Lmax, 128), 49)
    q = _rand_bits((S, gamma + 1, Hq, 128), 50)
    case(f"verify longest first S={S} Hkv={Hkv} paged={paged}")
    if paged:
        n = (Lmax + 15) // 16
        table = g.permutation(S * n).reshape(S, n).astype(np.int32)
        kd, vd = paged_kv(list(k), list(v), table, S * n, 16)
        out = bd.bd_verify_attn(kd, vd, bf16_dev(q), i32_dev(lens), page_table=i32_dev(table), max_seq_len=Lmax)
    else:
        out = bd.bd_verify_attn(bf16_dev(k), bf16_dev(v), bf16_dev(q), i32_dev(lens))
    torch.cuda.synchronize()
    assert_close(bf16_host64(out), O.verify_attn(k, v, q, lens, gamma)[0], f"longest first S={S}")


@pytest.mark.parametrize("P", [16, 24])
@pytest.mark.parametrize("S,Hkv,shared", [(6, 2, "all"), (6, 2, "prefix"), (70, 1, "pairs"), (1, 2, "all"), (40, 8, "all")])
def test_verify_shared_pages(S, Hkv, shared, P):
    # sequences that share pages take another load policy; one that starts outside the pool has keys absent from it
    gamma, G, Lmax = 2, 2, 300
    g = np.random.default_rng(61)
    lens = [int(n) for n in g.integers(gamma + 1, Lmax + 1, S)]
    lens[-1] = Lmax
    n = (Lmax + P - 1) // P
    table = (np.arange(S * n) % (4 * n)).reshape(S, n).astype(np.int32)    # sequences 4 apart share every page
    if shared == "all":
        table[:] = g.permutation(n)
    elif shared == "prefix":
        table = g.permutation(S * n).reshape(S, n).astype(np.int32)
        table[1::2, :3] = table[1, :3]
        table[2, 0] = -1
    pool = int(table.max()) + 1
    kp, vp = _rand_bits((pool, Hkv, P, 128), 62), _rand_bits((pool, Hkv, P, 128), 63)
    q = _rand_bits((S, gamma + 1, Hkv * G, 128), 64)
    case(f"verify shared pages S={S} Hkv={Hkv} {shared} P={P}")
    out = bd.bd_verify_attn(bf16_dev(kp), bf16_dev(vp), bf16_dev(q), i32_dev(lens), page_table=i32_dev(table),
                            max_seq_len=Lmax)
    torch.cuda.synchronize()
    got = bf16_host64(out)
    for s in range(0, S, 1 if S <= 8 else 9):
        if table[s, 0] < 0:
            assert np.isfinite(got[s]).all()
            continue
        rows = [np.ascontiguousarray(np.moveaxis(x[table[s]], 1, 0)).reshape(1, Hkv, n * P, 128) for x in (kp, vp)]
        assert_close(got[s:s + 1], O.verify_attn(*rows, q[s:s + 1], [lens[s]], gamma)[0], f"shared pages s={s}")


@pytest.mark.parametrize("Lmax", [383, 384, 400])
@pytest.mark.parametrize("S,Hkv,paged", [(64, 5, False), (9, 32, False), (9, 32, True), (65, 4, False)])
def test_verify_longest_first_rule(S, Hkv, paged, Lmax):
    # the order is taken from 384 keys on; lengths from the shortest possible to beyond the layout (taken as Lmax)
    gamma = 2
    g = np.random.default_rng(Lmax)
    lens = [int(n) for n in g.choice([gamma + 1, 40, 257, Lmax - 1, Lmax], S)]
    k, v = _rand_bits((S, Hkv, Lmax, 128), 71), _rand_bits((S, Hkv, Lmax, 128), 72)
    q = _rand_bits((S, gamma + 1, Hkv, 128), 73)
    given = [n + 9 if n == Lmax else n for n in lens]
    case(f"verify longest first S={S} Hkv={Hkv} Lmax={Lmax} paged={paged}")
    if paged:
        n = (Lmax + 15) // 16
        table = g.permutation(S * n).reshape(S, n).astype(np.int32)
        kd, vd = paged_kv(list(k), list(v), table, S * n, 16)
        out = bd.bd_verify_attn(kd, vd, bf16_dev(q), i32_dev(given), page_table=i32_dev(table), max_seq_len=Lmax)
    else:
        out = bd.bd_verify_attn(bf16_dev(k), bf16_dev(v), bf16_dev(q), i32_dev(given))
    torch.cuda.synchronize()
    assert_close(bf16_host64(out), O.verify_attn(k, v, q, lens, gamma)[0], f"longest first S={S} Lmax={Lmax}")


@pytest.mark.parametrize("V,ld,L", [
    (1, 900, 3196), (1, 900, 3197),      # the backward's table filled to the entry by one workgroup; one more: two
    (0, 0, 4063), (0, 0, 4064),          # the forward's, one branch
    (4, 1, 3930), (4, 1, 3931),          # the forward's with five branches, four of them a padded tile for one entry
])
def test_block_tables_filled(V, ld, L):
    # 256 units (8 sequences x 8 KV heads x 4 row groups): one workgroup takes a unit's whole stream if it can hold it
    S, Hkv, G, C = 8, 8, 4, 256
    lens = [L] * S
    k, v = _rand_bits((S, Hkv, L, 128), 310), _rand_bits((S, Hkv, L, 128), 311)
    qb = _rand_bits((S, C, Hkv * G, 128), 312)
    g = np.random.default_rng(313)
    idx_v = nsel_v = None
    if V:
        idx_v = np.stack([np.sort(g.choice(L, ld, replace=False)) for _ in range(V * S * Hkv)])
        idx_v = idx_v.reshape(V, S, Hkv, ld).astype(np.int32)
        nsel_v = np.full((V, S), ld, np.int32)
    _run(k, v, qb, idx_v, nsel_v, lens, f"filled V={V} ld={ld} L={L}", seqs=[7], seed=8)


@pytest.mark.parametrize("Hkv,C,V,ld,L", [(1, 16, 1, 32, 256), (2, 32, 1, 128, 1024), (1, 1, 0, 0, 32), (1, 1, 0, 0, 33),
                                          (4, 40, 1, 1, 64), (1, 16, 2, 31, 7)])
def test_backward_short_streams(Hkv, C, V, ld, L):
    # as many workgroups as the stream has tiles, one and two tiles, lists shorter than the stream that was planned.
    # Some row sees two keys or more: over a single key dQ is exactly zero, and the tolerance, a fraction of the
    # largest gradient, has nothing to hold the rounding of dP - D (128 fp32 products, about 1e-7) against.
    S, G = 2, 2
    lens = [L, max(1, L // 3)]
    k, v = _rand_bits((S, Hkv, L, 128), 320), _rand_bits((S, Hkv, L, 128), 321)
    qb = _rand_bits((S, C, Hkv * G, 128), 322)
    g = np.random.default_rng(323)
    idx_v = nsel_v = None
    if V:
        nsel_v = np.array([[min(ld, n) for n in lens]] * V, np.int32)
        idx_v = np.full((V, S, Hkv, ld), -1, np.int32)
        for i in range(V):
            for s in range(S):
                for h in range(Hkv):
                    idx_v[i, s, h, :nsel_v[i, s]] = np.sort(g.choice(lens[s], nsel_v[i, s], replace=False))
    _run(k, v, qb, idx_v, nsel_v, lens, f"short stream Hkv={Hkv} C={C} V={V} ld={ld} L={L}", seed=9)
