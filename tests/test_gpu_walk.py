"""The acceptance walk at the ends of its range: paths of 0, 1, 63 and all 64 nodes accepted, the
accepted path at the highest node indices, equally deep paths (lowest index wins) and duplicate
siblings - drafts are the target's own greedy tokens, so the expected path is known exactly."""
import numpy as np
import pytest

import workloads as wl
from paper_2604_13519_amd import binding as B
import gpu_utils as U

pytestmark = pytest.mark.gpu


def _greedy(model, cfg, K, V, root, n):
    kv = B.ts_kv_alloc(model, K.shape[1] + n + 80)
    B.ts_kv_import(kv, K, V)
    B.ts_set_pending(kv, root)
    out = []
    for _ in range(n):
        out.append(B.ts_verify(model, kv, [], [])[3])
        B.ts_kv_commit(kv)
    B.ts_kv_free(kv)
    return out


@pytest.mark.parametrize("accepted", [0, 1, 63, 64])
def test_walk_depths(accepted):
    cfg, w, model, om = U.get_model("micro_fp32")
    K, V = wl.gen_context_kv(cfg, 40, seed=9)
    g = _greedy(model, cfg, K, V, 5, 65)
    wrong = lambda t: (t + 1) % cfg.vocab  # noqa: E731
    kv = B.ts_kv_alloc(model, 200)
    B.ts_kv_import(kv, K, V)
    B.ts_set_pending(kv, 5)
    # one chain, wrong from node `accepted` on
    tok = [t if i < accepted else wrong(t) for i, t in enumerate(g[:64])]
    res = B.ts_verify(model, kv, tok, list(range(-1, 63)))
    assert res == (accepted, g[:accepted], list(range(accepted)), g[accepted])
    # the same path behind a block of rejected children of the root: it ends at the highest indices
    n = 64 - min(accepted, 32)
    k = 64 - n
    tok = [wrong(g[0])] * n + g[:k]
    par = [-1] * n + [-1] + list(range(n, 63)) if k else [-1] * n
    res = B.ts_verify(model, kv, tok, par)
    assert res == (k, g[:k], list(range(n, 64))[:k], g[k])
    # two equally deep copies of a path (duplicate siblings all along): the lower indices win
    d = max(1, accepted // 2)
    tok, par = [], []
    for i in range(d):
        tok += [g[i], g[i]]
        par += [2 * i - 2, 2 * i - 1] if i else [-1, -1]
    res = B.ts_verify(model, kv, tok, par)
    assert res == (d, g[:d], [2 * i for i in range(d)], g[d])
    B.ts_kv_free(kv)
