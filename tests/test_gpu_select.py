"""GPU parity of bd_select_kv.

Indices are integers, so parity is exact, in two parts:
  (i) the top-B stage is exact: the oracle's pooling and ranking applied to
      the GPU's own fp32 scores reproduces the GPU indices bit for bit;
 (ii) end to end the GPU indices equal the oracle's, except where the
      oracle's pooled scores at the selection boundary lie within a relative
      1e-4 of each other -- there fp32 and fp64 scores may legitimately rank
      two candidates differently; such boundaries are counted and every
      other position must agree.
Inputs whose scores are exact in any precision (all-zero keys) must agree
exactly end to end.
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2606_00144_amd as bd
import synth
from gpu_utils import bf16_dev, case, config_data, i32_dev, paged_kv

pytestmark = pytest.mark.gpu
DELTA = 1e-4


def _run_select(k, q_win, lens, Hq, W, B, page_table=None, kdev=None, **kw):
    case(f"select B={B} W={W} lens={list(lens)[:4]}")
    kd = bf16_dev(k) if kdev is None else kdev
    idx, nsel, scores = bd.bd_select_kv(kd, bf16_dev(q_win), i32_dev(lens), B, return_scores=True,
                                        page_table=page_table, **kw)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), nsel.cpu().numpy(), scores.cpu().numpy()


def _check(k, q_win, lens, Hq, W, B, what, pool_kernel=7, **kw):
    gi, gn, gs = _run_select(k, q_win, lens, Hq, W, B, pool_kernel=pool_kernel, **kw)
    oi, on, oraw = O.select_kv(k, q_win, lens, Hq, W, B, pool_kernel=pool_kernel)
    assert np.array_equal(gn, on), what
    S, Hkv = gi.shape[:2]
    near = 0
    for s in range(S):
        L = int(lens[s])
        for g in range(Hkv):
            if B >= L:
                assert np.array_equal(gi[s, g], oi[s, g]), (what, s, g)
                continue
            # (i) exact top-B on the GPU's own scores
            sel, _ = O.topk_from_scores(gs[s, g, :L].astype(np.float64), L, W, B, pool_kernel=pool_kernel)
            assert np.array_equal(gi[s, g], sel), (what, "top-B stage", s, g)
            # raw scores: each row sums to 1, so the total is W*G
            G = Hq // Hkv
            np.testing.assert_allclose(gs[s, g, :L].sum(dtype=np.float64), W * G, rtol=1e-4)
            np.testing.assert_allclose(gs[s, g, :L], oraw[s][g], rtol=1e-3, atol=1e-6)
            # (ii) end to end, differences only inside the near-tie band
            diff = set(gi[s, g].tolist()) ^ set(oi[s, g].tolist())
            if diff:
                pooled = O.max_pool(oraw[s][g][:L - W], pool_kernel)
                thr = np.sort(pooled)[::-1][B - W - 1]
                for t in diff:
                    assert abs(pooled[t] - thr) <= DELTA * thr, (what, s, g, t, pooled[t], thr)
                near += 1
    return near


def test_select_tiny4k():
    cfg = synth.workload("tiny-4k-gqa4")
    qt, k, v = config_data("tiny-4k-gqa4")
    near = _check(k, qt[:, -cfg.window:], [cfg.seq_len], cfg.num_q_heads, cfg.window, 256, "tiny 4K")
    assert near <= 1


@pytest.mark.parametrize("B", [256, 512, 1024, 2048])
def test_select_layer8k_budgets(B):
    cfg = synth.workload("llama3-8b-layer-8k")
    qt, k, v = config_data("llama3-8b-layer-8k")
    near = _check(k, qt[:, -cfg.window:], [cfg.seq_len], cfg.num_q_heads, cfg.window, B, f"8K layer B={B}")
    assert near <= 2


@pytest.mark.parametrize("pool_kernel", [1, 3, 5, 7, 9])
def test_select_pool_kernels(pool_kernel):
    # every pooling path of the top-B kernel: register windows (radius 0..3) and the general loop
    S, Hkv, Hq, W = 2, 2, 8, 32
    lens = [3000, 1337]
    g = np.random.default_rng(7)
    k = synth.f32_to_bf16_bits(g.standard_normal((S, Hkv, max(lens), 128)).astype(np.float32))
    q = synth.f32_to_bf16_bits(g.standard_normal((S, W, Hq, 128)).astype(np.float32))
    near = _check(k, q, lens, Hq, W, 300, f"pool {pool_kernel}", pool_kernel=pool_kernel)
    assert near <= 1


def test_select_longest_prefix():
    # L - W = BD_SELECT_MAX_PREFIX = 32768 prefix positions: every candidate slot of the top-B kernel
    # (32 per thread) and both ends of its staged range, beside a shorter sequence
    Hkv, Hq, W = 1, 4, 32
    lens = [32768 + W, 20000]
    g = np.random.default_rng(8)
    k = synth.f32_to_bf16_bits(g.standard_normal((2, Hkv, max(lens), 128)).astype(np.float32))
    q = synth.f32_to_bf16_bits(g.standard_normal((2, W, Hq, 128)).astype(np.float32))
    near = _check(k, q, lens, Hq, W, 2048, "prefix 32768")
    assert near <= 1


def test_select_zero_keys_exact_and_identity():
    S, Hkv, Hq, L, W = 2, 2, 8, 700, 16
    q = synth.f32_to_bf16_bits(np.random.default_rng(1).standard_normal((S, W, Hq, 128)).astype(np.float32))
    k = np.zeros((S, Hkv, L, 128), np.uint16)
    lens = [700, 300]
    gi, gn, gs = _run_select(k, q, lens, Hq, W, 400)
    oi, on, _ = O.select_kv(k, q, lens, Hq, W, 400)
    assert np.array_equal(gi, oi) and np.array_equal(gn, on)
    assert gn.tolist() == [400, 300]
    assert np.all(gi[1, :, 300:] == -1)
    assert gi[0, 0, :384].tolist() == list(range(384))


def test_select_lse_input_matches_two_pass():
    S, Hkv, Hq, L, W = 2, 2, 8, 1000, 32
    g = np.random.default_rng(2)
    k = synth.f32_to_bf16_bits(g.standard_normal((S, Hkv, L, 128)).astype(np.float32))
    q = synth.f32_to_bf16_bits(g.standard_normal((S, W, Hq, 128)).astype(np.float32))
    # fp64 log-sum-exp of each window row over its causal range
    sc = float(np.float32(1 / np.sqrt(128)))
    kf, qf = O.bf16_to_f64(k), O.bf16_to_f64(q)
    lse = np.zeros((S, W, Hq), np.float32)
    for s in range(S):
        for i in range(W):
            p = L - W + i
            for h in range(Hq):
                lg = sc * kf[s, h // 4, :p + 1] @ qf[s, i, h]
                lse[s, i, h] = np.logaddexp.reduce(lg)
    a = _run_select(k, q, [L, L], Hq, W, 200)
    case("select with lse_win")
    idx, nsel, scores = bd.bd_select_kv(bf16_dev(k), bf16_dev(q), i32_dev([L, L]), 200, return_scores=True,
                                        lse_win=torch.from_numpy(lse).cuda())
    torch.cuda.synchronize()
    np.testing.assert_allclose(scores.cpu().numpy(), a[2], rtol=1e-4, atol=1e-7)
    _check(k, q, [L, L], Hq, W, 200, "two-pass")


@pytest.mark.parametrize("Hq,Hkv,W", [(8, 8, 16), (4, 2, 4), (2, 2, 1)])
def test_select_one_row_tile(Hq, Hkv, W):
    # W * G <= 16 observation rows per KV head: the one-row-tile scoring path (padded rows see no key)
    S = 2
    lens = [2500, 777]
    g = np.random.default_rng(31 + W)
    k = synth.f32_to_bf16_bits(g.standard_normal((S, Hkv, max(lens), 128)).astype(np.float32))
    q = synth.f32_to_bf16_bits(g.standard_normal((S, W, Hq, 128)).astype(np.float32))
    near = _check(k, q, lens, Hq, W, 200, f"one row tile Hq={Hq} Hkv={Hkv} W={W}")
    assert near <= 1


def test_select_lse_input_indices_match_the_oracle():
    # the one-pass variant (the caller gives each window row's log-sum-exp) on the 8K layer: its indices
    # under the same two-part protocol as the two-pass selection
    cfg = synth.workload("llama3-8b-layer-8k")
    qt, k, _ = config_data("llama3-8b-layer-8k")
    W, L, Hq, G = cfg.window, cfg.seq_len, cfg.num_q_heads, cfg.num_q_heads // cfg.num_kv_heads
    qw = np.ascontiguousarray(qt[:, -W:])
    sc = float(np.float32(1 / np.sqrt(128)))
    kf, qf = O.bf16_to_f64(k[0]), O.bf16_to_f64(qw[0])
    lse = np.zeros((1, W, Hq), np.float32)
    for h in range(Hq):
        lg = sc * (qf[:, h] @ kf[h // G].T)                        # [W][L]
        for i in range(W):
            lse[0, i, h] = np.logaddexp.reduce(lg[i, :L - W + i + 1])
    for B in (256, 1024):
        near = _check(k, qw, [L], Hq, W, B, f"lse input B={B}", lse_win=torch.from_numpy(lse).cuda())
        assert near <= 2


def test_select_ragged_paged_mha():
    cfg = synth.workload("ragged-paged-b64-mha")
    lens = synth.seq_lens(cfg)[:4]
    ks, vs, qw = [], [], []
    for s in range(4):
        qt = synth.query_tail(cfg, s)
        kk, vv = synth.kv_sequence(cfg, s, q_tail=qt)
        ks.append(kk), vs.append(vv), qw.append(qt[-cfg.window:])
    table, npages = synth.page_table(cfg, lens)
    kd, _ = paged_kv(ks, vs, table, npages, cfg.page_size)
    near = _check(ks, np.stack(qw), lens, cfg.num_q_heads, cfg.window, 1024, "ragged paged paged",
                  page_table=i32_dev(table), kdev=kd)
    assert near <= 4


@pytest.mark.parametrize("L,at", [(40, 3), (40, 30), (300, 17), (1033, 700), (4097, 4000)])
def test_row_with_an_infinite_logit(L, at):
    # One window row's product with one key overflows.  The row's weight belongs to that key, whose score is not a
    # number; the row gives every other key nothing, and the other rows score as if it were not there.
    W, G, Hkv, B = 4, 2, 2, 16
    g = np.random.default_rng(77)
    q = g.standard_normal((1, W, Hkv * G, 128)).astype(np.float32)
    k = g.standard_normal((1, Hkv, L, 128)).astype(np.float32)
    q[..., 5] = 0.0
    q[0, 1, ::G, 5] = 100.0                      # window row 1, first query head of each KV head
    k[..., 5] = 0.0
    k[0, :, at, 5] = 3.0e38
    qb, kb = synth.f32_to_bf16_bits(q), synth.f32_to_bf16_bits(k)
    case(f"select infinite logit L={L} at={at}")
    _, _, sc = bd.bd_select_kv(bf16_dev(kb), bf16_dev(qb), i32_dev([L]), B, return_scores=True)
    torch.cuda.synchronize()
    got = sc.cpu().numpy().astype(np.float64)[0]
    qf, kf = O.bf16_to_f64(qb)[0], O.bf16_to_f64(kb)[0]
    for h in range(Hkv):
        want = np.zeros(L)
        for i in range(W):
            for j in range(G):
                if (i, j) == (1, 0):
                    continue
                n = L - W + i + 1                # keys that row i sees
                z = kf[h, :n] @ qf[i, h * G + j] / np.sqrt(128.0)
                p = np.exp(z - z.max())
                want[:n] += p / p.sum()
        others = np.arange(L) != at
        np.testing.assert_allclose(got[h, others], want[others], rtol=1e-3, atol=1e-6)
        assert not np.isfinite(got[h, at])
