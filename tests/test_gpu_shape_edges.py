"""Projection shapes at the edges of what the planner picks from: inner sizes of one and two 128-wide
chunks (shorter than every prefetch ring), column counts that leave a column group nearly empty,
row counts around the 16-row tiles (their padding rows come from a spare row) - and passes of more
than 80 rows over odd models, whose merge and cache write take the many-row kernels.  Against
the oracle, with the tolerances of the other parity tests."""
import numpy as np
import pytest

import workloads as wl
from oracle import toolspec_oracle as O
from paper_2604_13519_amd import binding as B
import gpu_utils as U

pytestmark = pytest.mark.gpu


def _load(**kw):
    cfg = wl.get_config("small_bf16").with_(name="shape_edges", **kw)
    w = wl.gen_weights(cfg, 21)
    model = B.ts_model_load(cfg, w)
    B.ts_model_keep_logits(model, True)
    return cfg, w, model, O.OracleModel(cfg, w, cache=True)


@pytest.mark.parametrize("kw", [
    dict(n_layers=2, d_model=128, n_q_heads=2, n_kv_heads=1, head_dim=64, d_ffn=128, vocab=31),     # every K one chunk
    dict(n_layers=2, d_model=256, n_q_heads=2, n_kv_heads=2, head_dim=128, d_ffn=384, vocab=2081),  # 2 and 3 chunks, one column past 65 groups
    dict(n_layers=1, d_model=640, n_q_heads=8, n_kv_heads=1, head_dim=64, d_ffn=1152, vocab=97),    # 5 and 9 chunks, 8 heads per KV head
])
def test_projection_shapes(kw):
    cfg, w, model, om = _load(**kw)
    rng = np.random.default_rng(3)
    for n, P in ((0, 33), (15, 16), (16, 130), (48, 64), (64, 65)):
        K, V = wl.gen_context_kv(cfg, P, seed=70 + n)
        kv, okv = U.make_pair(cfg, model, K, V, int(rng.integers(cfg.vocab)))
        tok, par = wl.random_tree(n, cfg.vocab, rng)
        U.check_verify(cfg, model, om, kv, okv, tok, par, label="d%d n%d P%d" % (cfg.d_model, n, P))
        B.ts_kv_free(kv)
    B.ts_model_free(model)


@pytest.mark.parametrize("hd,hq,hkv,n_seqs", [(64, 16, 4, 5), (128, 16, 2, 9)])
def test_many_rows_equal_single_passes(hd, hq, hkv, n_seqs):
    """Batches past 80 rows (and past 4096 (row, head) slots): rows of a ragged batch against the same
    requests alone, logits within the canary and cache rows within one-step flips."""
    cfg, w, model, om = _load(n_layers=2, d_model=256, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ffn=512, vocab=515)
    rng = np.random.default_rng(hd)
    nodes = [64 - (i % 3) for i in range(n_seqs)]
    lens = [3 + 61 * i for i in range(n_seqs)]
    trees = [wl.random_tree(n, cfg.vocab, rng) for n in nodes]
    kvs, ctx = [], []
    for i in range(n_seqs):
        K, V = wl.gen_context_kv(cfg, lens[i], seed=300 + i)
        kv = B.ts_kv_alloc(model, lens[i] + 70)
        B.ts_kv_import(kv, K, V)
        B.ts_set_pending(kv, i)
        kvs.append(kv)
    B.ts_verify_batch(model, kvs, trees)
    rows = sum(nodes) + n_seqs
    both = B.ts_get_logits(model, 0, rows, cfg.vocab)
    cache = [B.ts_kv_export(kv, lens[i], nodes[i] + 1, cfg) for i, kv in enumerate(kvs)]
    r0 = 0
    for i, kv in enumerate(kvs):
        B.ts_verify(model, kv, *trees[i])
        one = B.ts_get_logits(model, 0, nodes[i] + 1, cfg.vocab)
        assert U.rel_l2(both[r0:r0 + nodes[i] + 1], one) <= U.TOL_BF16_R
        k1, v1 = B.ts_kv_export(kv, lens[i], nodes[i] + 1, cfg)
        for a, b in ((cache[i][0], k1), (cache[i][1], v1)):
            assert U.rel_l2(wl.bf16_bits_to_f32(a), wl.bf16_bits_to_f32(b)) <= U.TOL_BF16_R
        r0 += nodes[i] + 1
        B.ts_kv_free(kv)
    B.ts_model_free(model)


@pytest.mark.parametrize("kw", [
    dict(d_model=1024, n_q_heads=8, n_kv_heads=2, vocab=32003),    # the head: 251 column groups, not a multiple of the XCDs
    dict(d_model=2048, n_q_heads=64, n_kv_heads=16, vocab=97),     # QKV: 96 column groups x 2 splits of eight chunks
])
def test_places_of_five_row_tiles(kw):
    """65 rows, one k-wave and a long K range: these launches leave the runs per XCD for round robin."""
    cfg, w, model, om = _load(n_layers=1, head_dim=128, d_ffn=256, **kw)
    rng = np.random.default_rng(kw["vocab"])
    K, V = wl.gen_context_kv(cfg, 40, seed=41)
    kv, okv = U.make_pair(cfg, model, K, V, 5)
    tok, par = wl.random_tree(64, cfg.vocab, rng)
    U.check_verify(cfg, model, om, kv, okv, tok, par, label="d%d" % cfg.d_model)
    B.ts_kv_free(kv)
    B.ts_model_free(model)


@pytest.mark.parametrize("n_seqs,P", [(4, 400), (4, 1950), (5, 1950)])
def test_merge_of_a_batch(n_seqs, P):
    """Joining key splits at both sides of the rule: 4160 (row, head) slots with up to eight splits and 5200
    with sixteen take a thread per 8 dims, 4160 with sixteen a workgroup per slot.  Against single passes."""
    cfg, w, model, om = _load(n_layers=1, d_model=256, n_q_heads=16, n_kv_heads=2, head_dim=128, d_ffn=256, vocab=97)
    rng = np.random.default_rng(P + n_seqs)
    trees, kvs = [wl.random_tree(64, cfg.vocab, rng) for _ in range(n_seqs)], []
    for i in range(n_seqs):
        K, V = wl.gen_context_kv(cfg, P + i, seed=700 + i)
        kvs.append(B.ts_kv_alloc(model, P + i + 65))
        B.ts_kv_import(kvs[i], K, V)
        B.ts_set_pending(kvs[i], i)
    B.ts_verify_batch(model, kvs, trees)
    both = B.ts_get_logits(model, 0, 65 * n_seqs, cfg.vocab).reshape(n_seqs, 65, cfg.vocab)
    for i, kv in enumerate(kvs):
        B.ts_verify(model, kv, *trees[i])
        one = B.ts_get_logits(model, 0, 65, cfg.vocab)
        assert max(U.rel_l2(a, b) for a, b in zip(both[i], one)) <= U.TOL_BF16_R
        B.ts_kv_free(kv)
    B.ts_model_free(model)


@pytest.mark.parametrize("d_model,hq,d_ffn", [
    (128, 1, 128),       # K of two chunks: less than the ring of the one-row-tile kernel holds
    (384, 3, 1152),      # six and eighteen chunks: exactly one round of the ring, and three
    (640, 5, 896),       # ten and fourteen: rests of four and two
    (1024, 8, 2944),     # K splits, 46 chunks
])
def test_one_and_two_row_tiles(d_model, hq, d_ffn):
    """Passes of one, fifteen, sixteen, seventeen and thirty-two rows: one row tile, two, and two with a single row."""
    cfg, w, model, om = _load(n_layers=1, d_model=d_model, n_q_heads=hq, n_kv_heads=hq, head_dim=128, d_ffn=d_ffn, vocab=1003)
    rng = np.random.default_rng(d_model + 1)
    K, V = wl.gen_context_kv(cfg, 70, seed=43)
    for n in (0, 14, 15, 16, 31):
        kv, okv = U.make_pair(cfg, model, K, V, 9)
        tok, par = wl.random_tree(n, cfg.vocab, rng)
        U.check_verify(cfg, model, om, kv, okv, tok, par, label="d%d rows %d" % (d_model, n + 1))
        B.ts_kv_free(kv)
    B.ts_model_free(model)


@pytest.mark.parametrize("d_model,hq,d_ffn,vocab,n_seqs,n_nodes", [
    (128, 1, 128, 97, 2, 40),        # 82 rows; every projection one chunk of 128
    (384, 3, 640, 1500, 3, 32),      # 99 rows; one chunk a split, gate/up and head three
    (256, 2, 1152, 5000, 2, 64),     # 130 rows, nine row tiles; one to three chunks
    (640, 5, 384, 8209, 4, 64),      # 260 rows, six row tiles in the head, which ends inside a tile
    (512, 4, 1536, 700, 7, 64),      # 455 rows; one to four chunks
    (1152, 9, 8064, 20011, 16, 64),  # 1040 rows; one k-wave (gate/up, head) and two (QKV, O, down), long ranges with rests
])
def test_many_rows_rings_and_small_heads(d_model, hq, d_ffn, vocab, n_seqs, n_nodes):
    """Passes of more than 80 rows over short and odd K ranges, and heads of few column groups.  Logits against single
    passes; the fused arg-max against the stored logits.  (Every variant of the kernel by itself, and ties between equal
    columns: test_gpu_projection_variants.py.)"""
    cfg, w, model, om = _load(n_layers=1, d_model=d_model, n_q_heads=hq, n_kv_heads=hq, head_dim=128, d_ffn=d_ffn, vocab=vocab)
    rng = np.random.default_rng(d_model)
    trees, kvs = [wl.random_tree(n_nodes, cfg.vocab, rng) for _ in range(n_seqs)], []
    for i in range(n_seqs):
        K, V = wl.gen_context_kv(cfg, 30 + i, seed=800 + i)
        kvs.append(B.ts_kv_alloc(model, 31 + i + n_nodes))
        B.ts_kv_import(kvs[i], K, V)
        B.ts_set_pending(kvs[i], i)
    rows = n_nodes + 1
    B.ts_verify_batch(model, kvs, trees)
    both = B.ts_get_logits(model, 0, rows * n_seqs, cfg.vocab)
    assert np.array_equal(B.ts_get_row_tokens(model, 0, rows * n_seqs), both.argmax(1))
    for i, kv in enumerate(kvs):
        B.ts_verify(model, kv, *trees[i])
        one = B.ts_get_logits(model, 0, rows, cfg.vocab)
        assert max(U.rel_l2(a, b) for a, b in zip(both[i * rows:(i + 1) * rows], one)) <= U.TOL_BF16_R, "sequence %d" % i
        B.ts_kv_free(kv)
    B.ts_model_free(model)


@pytest.mark.parametrize("contexts,n_nodes,hq,hd", [
    ((2600, 150), 20, 8, 128),                          # two sequences, few KV heads: more than 16 splits, and three
    ((0, 63, 64, 1900, 700), 64, 16, 128),              # two blocks, two and three, and the longest 31: ragged splits, many slots
    ((0, 61, 62, 2600), 2, 8, 128),                     # three keys, exactly one block and one key more beside 41 blocks
    (tuple(40 + 9 * i for i in range(130)), 2, 8, 128),  # more sequences than one round of workgroups holds
    ((0, 61, 62, 2600), 2, 8, 64),                      # heads of 64: merged by a workgroup per slot
    ((0, 63, 64, 1900, 700, 1200), 64, 16, 64),         # ... and by a thread per 8 dims
])
def test_units_of_a_ragged_batch(contexts, n_nodes, hq, hd):
    """Key blocks dealt to workgroups in proportion to the lengths of a batch.  Against single passes."""
    cfg, w, model, om = _load(n_layers=1, d_model=256, n_q_heads=hq, n_kv_heads=2, head_dim=hd, d_ffn=256, vocab=97)
    rng = np.random.default_rng(len(contexts))
    trees, kvs = [wl.random_tree(n_nodes, cfg.vocab, rng) for _ in contexts], []
    for i, P in enumerate(contexts):
        kvs.append(B.ts_kv_alloc(model, P + n_nodes + 1))
        if P:
            K, V = wl.gen_context_kv(cfg, P, seed=900 + i)
            B.ts_kv_import(kvs[i], K, V)
        B.ts_set_pending(kvs[i], i % cfg.vocab)
    rows = n_nodes + 1
    B.ts_verify_batch(model, kvs, trees)
    both = B.ts_get_logits(model, 0, rows * len(contexts), cfg.vocab).reshape(len(contexts), rows, cfg.vocab)
    for i, kv in enumerate(kvs):
        B.ts_verify(model, kv, *trees[i])
        one = B.ts_get_logits(model, 0, rows, cfg.vocab)
        assert max(U.rel_l2(a, b) for a, b in zip(both[i], one)) <= U.TOL_BF16_R, "sequence %d" % i
        B.ts_kv_free(kv)
    B.ts_model_free(model)


def test_partials_of_one_long_request_among_many():
    """Key splits of one long request cost room for its own rows, not for those of the 400 short ones beside it:
    13 splits for all 6817 rows would be 374 MB, for its 17 rows they are 29 MB.  Rows against single passes."""
    import torch
    cfg, w, model, om = _load(n_layers=1, d_model=256, n_q_heads=16, n_kv_heads=2, head_dim=128, d_ffn=256, vocab=97)
    rng = np.random.default_rng(5)
    n_seqs, nodes, long_one = 401, 16, 200
    trees = [wl.random_tree(nodes, cfg.vocab, rng) for _ in range(n_seqs)]
    kvs = []
    for i in range(n_seqs):
        K, V = wl.gen_context_kv(cfg, 20 + i % 7, seed=1000 + i)
        kvs.append(B.ts_kv_alloc(model, 4200 if i == long_one else 60))
        B.ts_kv_import(kvs[i], K, V)
        B.ts_set_pending(kvs[i], i % cfg.vocab)
    B.ts_verify_batch(model, kvs, trees)                   # the workspace of as many rows, short contexts only
    K, V = wl.gen_context_kv(cfg, 4160, seed=77)
    B.ts_kv_import(kvs[long_one], K, V)
    before = torch.cuda.mem_get_info()[0]
    B.ts_verify_batch(model, kvs, trees)
    grown = before - torch.cuda.mem_get_info()[0]
    assert grown <= 32 << 20, "the pass took %.0f MB more" % (grown / 1e6)
    rows = nodes + 1
    both = B.ts_get_logits(model, 0, rows * n_seqs, cfg.vocab).reshape(n_seqs, rows, cfg.vocab)
    for i in (0, 1, long_one - 1, long_one, long_one + 1, n_seqs - 1):
        B.ts_verify(model, kvs[i], *trees[i])
        one = B.ts_get_logits(model, 0, rows, cfg.vocab)
        assert max(U.rel_l2(a, b) for a, b in zip(both[i], one)) <= U.TOL_BF16_R, "sequence %d" % i
    for kv in kvs:
        B.ts_kv_free(kv)
    B.ts_model_free(model)


@pytest.mark.parametrize("hq,hkv", [(2, 2), (4, 2), (8, 2)])
def test_row_tiles_of_one_wave(hq, hkv):
    """One, two and three 16-row tiles in a wave (more rows take two waves) with one, two and four query heads per
    KV head, which is one wave each: the smallest workgroups stage the most vectors per thread, and three tiles walk a
    block's halves in a loop.  Contexts of one block, of several splits, and ending inside a half."""
    cfg, w, model, om = _load(n_layers=1, d_model=256, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, d_ffn=256, vocab=97)
    rng = np.random.default_rng(hq)
    for n, P in ((5, 700), (31, 20), (32, 333), (40, 1500), (47, 96)):
        K, V = wl.gen_context_kv(cfg, P, seed=500 + n)
        kv, okv = U.make_pair(cfg, model, K, V, int(rng.integers(cfg.vocab)))
        tok, par = wl.random_tree(n, cfg.vocab, rng)
        U.check_verify(cfg, model, om, kv, okv, tok, par, label="hq%d n%d P%d" % (hq, n, P))
        B.ts_kv_free(kv)
    B.ts_model_free(model)


def test_workspace_of_a_very_large_batch():
    """253 requests of 65 rows under a feed-forward of 131072 grow the workspace until a plane of the
    projection inputs (16480 + 80 rows, 4.3 GB) passes 32-bit offsets, and the batch's last row blocks lie beyond
    them as well.  Every request of the batch is the same, so its rows have to be the same to the bit; a single
    request afterwards runs the kernels it ran before, so its rows have to be what they were."""
    cfg = wl.get_config("small_bf16").with_(name="wide_ffn", n_layers=1, d_model=128, n_q_heads=1, n_kv_heads=1, head_dim=128,
                                            d_ffn=131072, vocab=64)
    model = B.ts_model_load(cfg, wl.gen_weights(cfg, 5))
    B.ts_model_keep_logits(model, True)
    n_seqs, nodes, P = 253, 64, 16
    assert (n_seqs * (nodes + 1) // 80 * 80 + 160) * cfg.d_ffn * 2 > 1 << 32
    tok, par = wl.random_tree(nodes, cfg.vocab, np.random.default_rng(9))
    K, V = wl.gen_context_kv(cfg, P, seed=31)
    pool = B.ts_kv_pool_create(model, n_seqs * ((P + nodes + 16) // 16))
    kvs = [B.ts_kv_alloc_pooled(pool, P + nodes + 1) for _ in range(n_seqs)]
    for kv in kvs:
        B.ts_kv_import(kv, K, V)
        B.ts_set_pending(kv, 3)

    def single():
        res = B.ts_verify(model, kvs[0], tok, par)
        return res, B.ts_get_logits(model, 0, nodes + 1, cfg.vocab)

    res, before = single()
    batch = B.ts_verify_batch(model, kvs, [(tok, par)] * n_seqs)
    rows = B.ts_get_logits(model, 0, n_seqs * (nodes + 1), cfg.vocab).reshape(n_seqs, nodes + 1, cfg.vocab)
    assert all(np.array_equal(rows[0], r) for r in rows[1:]) and all(b == batch[0] for b in batch)
    assert U.rel_l2(rows[0], before) <= U.TOL_BF16_R
    res_after, after = single()
    assert np.array_equal(before, after) and res_after == res
    for kv in kvs:
        B.ts_kv_free(kv)
    B.ts_kv_pool_free(pool)
    B.ts_model_free(model)
