"""The kinds that the profile summaries report, from kernel names in launch order: QKV, O and down run one
kernel whose shape and grid follow the planner, so only their place in the layer tells them apart."""
import sqlite3

import pytest

from paper_2604_13519_amd import counters as C


def _pass(partial, swiglu, head, attn, merge, layers=2):
    """(kernel, kind) of one verify pass in launch order"""
    seq = [("k_embed_rope<unsigned short>", "embed_rope_table")]
    for _ in range(layers):
        seq += [("k_norm<unsigned short>", "residual_rmsnorm"), (partial[0], "gemm_qkv"), ("k_rope_kv<unsigned short>", "rope_kv_write"),
                (attn, "attn_bf16"), (merge, "attn_merge"), (partial[1], "gemm_o"), ("k_norm<unsigned short>", "residual_rmsnorm"),
                (swiglu, "gemm_gate_up"), (partial[2], "gemm_down")]
    return seq + [("k_norm<unsigned short>", "residual_rmsnorm"), (head, "gemm_lm_head_argmax"), ("k_walk", "accept_walk")]


SKINNY = "k_gemm_bf16<5, 2, 8, 1, 128, 1, %d, 8>"
ROWS = "k_gemm_rows_bf16<%d, 8, 1, %d>"
ONE = _pass([SKINNY % 0] * 3, "k_gemm_bf16<5, 2, 4, 2, 128, 2, 2, 8>", SKINNY % 1, "k_attn_bf16<128, 3, 2, 4>", "k_attn_merge")
BATCH = _pass([ROWS % (5, 0), ROWS % (7, 0), ROWS % (5, 0)], ROWS % (4, 2), ROWS % (7, 1), "k_attn_bf16<128, 3, 0, 4>", "k_attn_merge_few")
LOAD = [("k_repack_tiles", None), ("__amd_rocclr_copyBuffer", None), ("k_kv_xfer<unsigned short, true>", None)]
SEQ = LOAD + ONE + [("k_commit<unsigned short>", None)] + BATCH + [("k_plain_read", "plain_read")] + ONE


def test_kinds_follow_the_place_in_the_layer():
    assert C.kernel_kinds([k for k, _ in SEQ]) == [kind for _, kind in SEQ]


def test_a_counter_pass_is_grouped_by_kind(tmp_path):
    db = str(tmp_path / "p.db")
    con = sqlite3.connect(db)
    con.execute("create table counters_collection (dispatch_id int, kernel_name text, counter_name text, value real)")
    for i, (k, _) in reversed(list(enumerate(SEQ))):        # the table is in no particular order
        con.execute("insert into counters_collection values (?, ?, 'X', ?)", (i, "void (anonymous namespace)::%s(GemmArgs)" % k, float(i)))
    con.commit()
    con.close()
    got = C._load(db)
    for kind in ("gemm_qkv", "gemm_o", "gemm_down", "attn_merge"):
        want = sorted(float(i) for i, (_, x) in enumerate(SEQ) if x == kind)
        assert sorted(v for k, c in got.items() if k[0] == kind for v in c["X"]) == want
    assert len([k for k in got if k[0] == "gemm_qkv"]) == 2 and sum(len(c["X"]) for c in got.values()) == len(SEQ)


@pytest.mark.parametrize("name,mode", [("k_gemm_bf16<1, 2, 4, 1, 128, 1, 0, 8>", 0), ("k_gemm_few_bf16<1, 1, 2, 4, 128, 4, 1>", 1), ("k_gemm_rows_bf16<8, 2, 4, 2>", 2),
                                       ("k_gemm_rows_bf16<4, 8, 1, 1>", 1), ("k_gemm_f32<1, 1, false>", None), ("k_norm<float>", None)])
def test_projection_modes(name, mode):
    assert C._gemm_mode(name) == mode
