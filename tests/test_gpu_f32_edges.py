"""fp32 path at the edges of its tiles: inner sizes that are no multiple of the 16-wide k chunk, row
counts around the 16 / 32 / 64-row tiles, ragged column tiles, every head_dim class of the
attention kernel, contexts around page edges - against the oracle (contract of the fp32 path)."""
import numpy as np
import pytest

import workloads as wl
from oracle import toolspec_oracle as O
from paper_2604_13519_amd import binding as B
import gpu_utils as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model,hq,hkv,hd,ffn,vocab", [
    (20, 3, 1, 8, 16, 37),        # K = 20, 24, 16: one chunk and a remainder of 4 and 8
    (36, 2, 2, 16, 48, 17),       # K = 36, 32, 48
    (100, 4, 2, 128, 144, 131),   # head_dim 128: two keys per wave, two page parts
    (132, 2, 1, 64, 272, 33),     # more chunks than one round of the 8 waves holds
])
def test_f32_tiles(d_model, hq, hkv, hd, ffn, vocab):
    cfg = wl.get_config("micro_fp32").with_(name="f32_edges", d_model=d_model, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd,
                                            d_ffn=ffn, vocab=vocab)
    w = wl.gen_weights(cfg, 7)
    model = B.ts_model_load(cfg, w)
    B.ts_model_keep_logits(model, True)
    om = O.OracleModel(cfg, w, cache=True)
    rng = np.random.default_rng(11)
    for n, P in ((0, 1), (15, 15), (16, 16), (32, 17), (64, 300), (31, 1100)):
        K, V = wl.gen_context_kv(cfg, P, seed=50 + n)
        kv, okv = U.make_pair(cfg, model, K, V, int(rng.integers(vocab)))
        tok, par = wl.random_tree(n, vocab, rng)
        U.check_verify(cfg, model, om, kv, okv, tok, par, label="f32 d%d hd%d n%d P%d" % (d_model, hd, n, P))
        B.ts_kv_free(kv)
    B.ts_model_free(model)


def test_f32_attention_at_its_largest_context():
    """15000 keys, the most the fp32 path takes (scores and page table of a row fill the LDS): the same
    tree one key further is refused."""
    cfg, w, model, om = U.get_model("micro_fp32")
    n, P = 9, 14990
    K, V = wl.gen_context_kv(cfg, P, seed=8)
    kv, okv = U.make_pair(cfg, model, K, V, 3, capacity=P + 20)
    tok, par = wl.random_tree(n, cfg.vocab, np.random.default_rng(1))
    U.check_verify(cfg, model, om, kv, okv, tok, par, label="f32 15000 keys")
    with pytest.raises(B.TsError) as e:
        B.ts_verify(model, kv, np.append(tok, 1), np.append(par, -1))
    assert e.value.status == B.TS_ERR_KV_CAPACITY
    B.ts_kv_free(kv)
