"""The calls a serving program makes of this framework, as measurable cases.

A program that serves tool-calling requests loads a model once (ts_model_load), keeps one paged
K/V cache per request, and then makes three kinds of calls, all of which are here through the
binding: ts_verify / ts_verify_batch on a draft tree (or on no draft at all: plain decoding),
ts_verify_sample for stochastic acceptance, and ts_prefill for prompts and tool results.  A pass is
one such call - for ingestion, the call and the first verification on top of it - and its outputs
are the logits of every row of the pass.

Model shapes are those of workloads/configs.py with fewer layers and, where the head is not what a
case is about, a small vocabulary: a verify pass is a chain of identical layers, so eight of them
behave like thirty-two, and the small vocabulary keeps the copy of the logits (which the shipped
greedy path never makes) a few per cent of the pass.  Weights are the program's checkpoint: fixed,
loaded once per process.  Everything that belongs to a request - context K/V, root token, tree,
prompt - comes from the case's seed.
"""
import ctypes
import math
import zlib

import numpy as np
import torch

import workloads as wl
from paper_2604_13519_amd import binding as B

F32 = wl.configs.DTYPE_F32
MODELS = {
    # workload 1 as it is: two fp32 layers, d 256
    "tiny_fp32": wl.get_config("tiny_fp32"),
    # the small bf16 shapes with three / two layers, ragged vocabulary, random norm gains
    "small": wl.get_config("small_bf16"),
    "small_hd64": wl.get_config("small_bf16_hd64"),
    # eight layers of the 8B shape (bench workloads w2, w3, w4, w6 and end to end)
    "8b": wl.get_config("llama8b").with_(name="8b", n_layers=8, vocab=8192, norm_init="random"),
    # one layer of the 8B shape under its full vocabulary: the head and the sampling step
    "8b_head": wl.get_config("llama8b").with_(name="8b_head", n_layers=1, norm_init="random"),
    # two layers of the 32B-class shape (bench workload w5)
    "32b": wl.get_config("qwen32b").with_(name="32b", n_layers=2, vocab=8192, norm_init="random"),
}

# call: verify (one request), batch, sample, prefill.  nodes: draft nodes per request (0 = plain
# decoding).  tree: builder in workloads/trees.py.  context: committed tokens; batches have ragged
# contexts between context / spread and context.  prompt: tokens ingested before the verification.
_BASE = {"call": "verify", "tree": "bfs", "requests": 1, "spread": 1, "prompt": 0, "paged": False}


def _case(name, model, context, nodes, **kw):
    return dict(_BASE, name=name, model=model, context=context, nodes=nodes, **kw)


def listed():
    return [
        # the smallest call: workload 1, a chain of 8 over 512 tokens in fp32; launches and latency
        _case("tiny_fp32_chain8", "tiny_fp32", 512, 8, tree="chain"),
        # a small bf16 draft model's step, odd context: launches and latency
        _case("small_tree25", "small", 733, 25),
        # plain decoding of an 8B-shaped model: what every step without a draft costs
        _case("8b_decode", "8b", 4096, 0),
        # bench w2: one retrieved continuation of 16 tokens
        _case("8b_chain16", "8b", 4096, 16, tree="chain"),
        # bench w3, the headline: schema chain, tool-name alternatives, argument chain, retrieved branches
        _case("8b_tree64", "8b", 8192, 64, tree="schema"),
        # a long agent history with an odd length and a tree that fills no tile
        _case("8b_tree37_long", "8b", 23011, 37),
        # bench w4: sixteen requests of a server, ragged contexts out of one page pool, 528 rows
        _case("8b_batch16", "8b", 8192, 32, call="batch", requests=16, spread=4, paged=True),
        # bench w5: four long requests of a 32B-class model, 260 rows
        _case("32b_batch4", "32b", 32768, 64, call="batch", requests=4, tree="schema"),
        # a tool result of odd length joins a conversation, then the next tree is verified
        _case("8b_prefill_333", "8b", 2000, 64, call="prefill", prompt=333, tree="schema"),
        # a fresh prompt (system text and tool documentation), then the first tree
        _case("8b_prefill_4096", "8b", 0, 64, call="prefill", prompt=4096, tree="schema"),
        # stochastic acceptance under the full vocabulary: the head and the sampling step
        _case("8b_head_sample8", "8b_head", 1024, 8, call="sample", tree="chain"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["tiny", "small", "verify", "verify", "batch", "batch32", "prefill", "sample"])
    tree = rng.choice(["bfs", "random", "chain"])
    if kind == "tiny":
        c = _case(None, "tiny_fp32", _log_int(rng, 32, 2048), rng.randint(0, 32), tree=tree)
    elif kind == "small":
        c = _case(None, rng.choice(["small", "small_hd64"]), _log_int(rng, 32, 8192), rng.randint(0, 64), tree=tree)
    elif kind == "verify":
        c = _case(None, "8b", _log_int(rng, 64, 23000), rng.randint(0, 64), tree=tree)
    elif kind == "batch":
        n = rng.randint(2, 16)
        c = _case(None, "8b", _log_int(rng, 256, 8192), rng.randint(0, 32), call="batch", requests=n,
                  spread=rng.randint(2, 6), tree=tree, paged=rng.random() < 0.5)
    elif kind == "batch32":
        c = _case(None, "32b", _log_int(rng, 512, 32768), rng.randint(4, 64), call="batch", requests=rng.randint(1, 4), tree=tree)
    elif kind == "prefill":
        c = _case(None, "8b", rng.choice([0, rng.randint(1, 4000)]), rng.randint(1, 64), call="prefill",
                  prompt=_log_int(rng, 40, 3500), tree=tree)
    else:
        c = _case(None, "8b_head", _log_int(rng, 64, 4096), rng.randint(0, 16), call="sample", tree=tree)
    del c["name"]
    return c


# ---- inputs ------------------------------------------------------------------------------------
def _gen(*key):
    g = torch.Generator(device="cuda")
    g.manual_seed(zlib.crc32(repr(key).encode()) + (1 << 33))
    return g


def _dtype(cfg):
    return torch.float32 if cfg.dtype == F32 else torch.bfloat16


def _weight(cfg, kind, layer=-1):
    """One tensor of the checkpoint on the GPU, in the storage type: N(0, 0.02), gains around 1."""
    x = torch.randn(wl.tensor_shapes(cfg)[kind], generator=_gen("weights", cfg.name, kind, layer), device="cuda")
    x = (1.0 + 0.1 * x) if kind.startswith("norm") and cfg.norm_init == "random" else torch.ones_like(x) if kind.startswith("norm") else 0.02 * x
    return x.to(_dtype(cfg))


def _host(x):
    x = x.contiguous()
    return x.cpu().numpy() if x.dtype == torch.float32 else x.view(torch.int16).cpu().numpy().view(np.uint16)


_models = {}


def _model(name):
    if name not in _models:
        cfg = MODELS[name]
        w = {k: _host(_weight(cfg, k)) for k in wl.weights.GLOBAL_KINDS}
        w["layers"] = [{k: _host(_weight(cfg, k, l)) for k in wl.weights.LAYER_KINDS} for l in range(cfg.n_layers)]
        m = B.ts_model_load(cfg, w)
        B.ts_model_keep_logits(m, True)
        _models[name] = m
    return _models[name]


def _contexts(case):
    """Committed length of every request: ragged between context / spread and context, the longest first."""
    n, hi = case["requests"], case["context"]
    lo = max(1, hi // case["spread"]) if hi else 0
    return [hi - (hi - lo) * i // max(1, n - 1) for i in range(n)]


def _context_kv(cfg, seed, request, n_pos):
    """Context K/V as the cache holds it: N(0, 1) in the storage type, [layers][positions][KV heads][head_dim]."""
    shape = (cfg.n_layers, n_pos, cfg.n_kv_heads, cfg.head_dim)
    g = _gen("kv", seed, request)
    return [torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(_dtype(cfg)) for _ in range(2)]


def _trees(case, cfg, seed):
    """Per request (root token, draft tokens, parents)."""
    rng, out = np.random.default_rng([seed, 77]), []
    for _ in range(case["requests"]):
        n = case["nodes"]
        if case["tree"] == "schema":
            tok, par = wl.schema_retrieval_tree([], cfg.vocab, rng)
        elif case["tree"] == "chain":
            tok, par = wl.chain_tree([], n, 0.0, cfg.vocab, rng)
        elif case["tree"] == "random" or n == 0:
            tok, par = wl.random_tree(n, cfg.vocab, rng)
        else:   # breadth first; a small branching factor needs a deeper tree to hold every node
            tok, par = wl.bfs_tree([], n, cfg.vocab, rng, max_depth=64)
        out.append((int(rng.integers(cfg.vocab)), tok[:n].astype(np.int32), par[:n].astype(np.int32)))
    return out


def _prompt(case, cfg, seed):
    return np.random.default_rng([seed, 78]).integers(cfg.vocab, size=case["prompt"]).astype(np.int32)


_staging = {}


def _pinned(slot, like):
    """The program's pinned staging buffer for cache imports: kept, grown when a request needs more."""
    n = like.numel() * like.element_size()
    if slot not in _staging or _staging[slot].numel() < n:
        _staging[slot] = torch.empty(n, dtype=torch.uint8, pin_memory=True)
    t = _staging[slot][:n].view(like.dtype).view(like.shape)
    t.copy_(like)
    return t.numpy() if t.dtype == torch.float32 else t.view(torch.int16).numpy().view(np.uint16)


class _State:
    """One program's requests: their caches, trees, prompt and the buffer it reads logits into."""

    def __init__(self, case, seed):
        cfg = self.cfg = MODELS[case["model"]]
        self.case, self.model, self.kvs, self.pool = case, _model(case["model"]), [], None
        self.ctx = _contexts(case)
        self.trees = _trees(case, cfg, seed)
        self.prompt = _prompt(case, cfg, seed)
        cap = [p + case["prompt"] + case["nodes"] + 1 for p in self.ctx]
        if case["paged"]:
            self.pool = B.ts_kv_pool_create(self.model, sum((c + 15) // 16 for c in cap))
        for i, p in enumerate(self.ctx):
            kv = B.ts_kv_alloc_pooled(self.pool, cap[i]) if case["paged"] else B.ts_kv_alloc(self.model, cap[i])
            self.kvs.append(kv)
            if p:
                k, v = _context_kv(cfg, seed, i, p)
                B.ts_kv_import(kv, _pinned("k", k), _pinned("v", v))
            B.ts_set_pending(kv, self.trees[i][0])
        rng = np.random.default_rng([seed, 79])
        self.uniform, self.noise = rng.random(case["nodes"], dtype=np.float32), int(rng.integers(1 << 62))
        self.rows = sum(len(t[1]) + 1 for t in self.trees)
        self.logits = torch.empty((self.rows, cfg.vocab), dtype=torch.float32, pin_memory=True)

    def __del__(self):
        try:
            for kv in self.kvs:
                B.ts_kv_free(kv)
            if self.pool is not None:
                B.ts_kv_pool_free(self.pool)
        except Exception:
            pass


def prepare(case, seed):
    return _State(case, seed)


def run(s):
    call = s.case["call"]
    if call == "prefill":
        # the conversation as it was, then the new text; its last token is the tree's root
        B.ts_kv_truncate(s.kvs[0], s.ctx[0])
        B.ts_set_pending(s.kvs[0], s.trees[0][0])
        B.ts_prefill(s.model, s.kvs[0], s.prompt)
    if call == "batch":
        B.ts_verify_batch(s.model, s.kvs, [t[1:] for t in s.trees])
    elif call == "sample":
        B.ts_verify_sample(s.model, s.kvs[0], s.trees[0][1], s.trees[0][2], 0.8, s.uniform, s.noise)
    else:
        B.ts_verify(s.model, s.kvs[0], s.trees[0][1], s.trees[0][2])
    st = B.load_library().ts_get_logits(s.model, 0, s.rows, ctypes.c_void_p(s.logits.data_ptr()))
    if st != B.TS_OK:
        raise B.TsError(st, "ts_get_logits")
    return s.logits


# ---- what a pass cannot do without ---------------------------------------------------------------
def work(case):
    cfg = MODELS[case["model"]]
    esz = 4 if cfg.dtype == F32 else 2
    per_layer = (cfg.streamed_params() - cfg.vocab * cfg.d_model) // cfg.n_layers
    layers, head = per_layer * cfg.n_layers, cfg.vocab * cfg.d_model
    rows = case["requests"] * (case["nodes"] + 1)
    n_bytes = esz * (layers + head) + 4 * rows * cfg.vocab
    flops = 2 * rows * (layers + head)
    for p in _contexts(case):
        total = p + case["prompt"]
        n_bytes += total * cfg.kv_bytes_per_token()
        flops += 4 * cfg.n_layers * cfg.q_dim * (case["nodes"] + 1) * total
    if case["prompt"]:       # the ingestion: its own pass over the layers, causal attention, K/V written
        n, p = case["prompt"], case["context"]
        n_bytes += esz * layers + (p + n) * cfg.kv_bytes_per_token()
        flops += 2 * n * layers + 4 * cfg.n_layers * cfg.q_dim * (n * p + n * n // 2)
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    """Four times what one request's logits differ by when its sums run in another order: the same
    request alone, inside batches of two and six, and with its prompt ingested in two pieces.
    Seen at most: 8B and 32B shapes rel 1.06e-3, max 4.5e-3 (a last-bit difference flips single bf16
    K/V entries, half queries and probabilities); small shapes rel 1.0e-4, max 1.0e-3 on one seed and
    twice that on others; fp32 rel 0.9e-6, max 4.0e-6 against 64 bits."""
    if MODELS[case["model"]].dtype == F32:
        return {"rel": 4e-6, "max": 2e-5}
    if case["model"].startswith("small"):
        return {"rel": 1e-3, "max": 8e-3}
    return {"rel": 4e-3, "max": 2e-2}


# ---- the same logits in 64 bits, plain torch --------------------------------------------------------
def _rms(x, gain, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * gain


def _rope(x, pos, theta):
    """x [rows][heads][hd]; pair (j, j + hd/2) rotated by pos * theta^(-2j/hd)."""
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * theta ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    cos, sin = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)


def _attend(q, K, V, see, scale):
    """q [rows][Hq][hd], K/V [keys][Hkv][hd], see [rows][keys]; a row sees the keys that see allows."""
    rows, hq, hd = q.shape
    hkv, out = K.shape[1], torch.empty_like(q)
    for h in range(hq):
        g = h // (hq // hkv)
        for r in range(0, rows, 512):
            s = (q[r:r + 512, h].contiguous() @ K[:, g].t().contiguous()) * scale
            s.masked_fill_(~see[r:r + 512], -math.inf)
            out[r:r + 512, h] = torch.softmax(s, -1) @ V[:, g].contiguous()
    return out


def exact(case, seed):
    cfg = MODELS[case["model"]]
    dev, hd = "cuda", cfg.head_dim
    prompt = _prompt(case, cfg, seed)
    seqs, r0 = [], 0
    for i, (p, (root, tok, par)) in enumerate(zip(_contexts(case), _trees(case, cfg, seed))):
        # rows: [root of the ingestion, prompt without its last token] (causal), then the tree under the pending token
        chain = [root] + prompt[:-1].tolist() if len(prompt) else []
        tree_root = int(prompt[-1]) if len(prompt) else root
        toks = chain + [tree_root] + tok.tolist()
        n, m = len(chain), len(tok) + 1
        depth, see_tree = np.zeros(m, np.int64), np.zeros((m, m), bool)
        see_tree[0, 0] = True
        for j in range(1, m):
            up = int(par[j - 1]) + 1
            depth[j] = depth[up] + 1
            see_tree[j] = see_tree[up]
            see_tree[j, j] = True
        see = torch.ones((n + m, p + n + m), dtype=torch.bool, device=dev)
        see[:n, p:] = torch.ones((n, n + m), dtype=torch.bool, device=dev).tril()
        see[n:, p + n:] = torch.from_numpy(see_tree).to(dev)
        pos = torch.cat([torch.arange(n), n + torch.from_numpy(depth)]).to(dev) + p
        k, v = _context_kv(cfg, seed, i, p) if p else (None, None)
        seqs.append((r0, n, m, p, toks, see, pos, k, v))
        r0 += n + m
    tok = torch.tensor(sum((s[4] for s in seqs), []), device=dev)
    pos = torch.cat([s[6] for s in seqs])
    h = _weight(cfg, "embed")[tok].double()
    mat = lambda x, kind, l: x @ _weight(cfg, kind, l).double().t()  # noqa: E731
    gain = lambda kind, l=-1: _weight(cfg, kind, l).double()  # noqa: E731
    for l in range(cfg.n_layers):
        x = _rms(h, gain("norm1", l), cfg.rms_eps)
        q = _rope(mat(x, "wq", l).view(-1, cfg.n_q_heads, hd), pos, cfg.rope_theta)
        k = _rope(mat(x, "wk", l).view(-1, cfg.n_kv_heads, hd), pos, cfg.rope_theta)
        v = mat(x, "wv", l).view(-1, cfg.n_kv_heads, hd)
        a = torch.empty_like(q)
        for r, n, m, p, _, see, _, ck, cv in seqs:
            sl = slice(r, r + n + m)
            K = torch.cat([ck[l].double(), k[sl]]) if p else k[sl]
            V = torch.cat([cv[l].double(), v[sl]]) if p else v[sl]
            a[sl] = _attend(q[sl], K, V, see, 1.0 / math.sqrt(hd))
        h = h + mat(a.reshape(len(tok), -1), "wo", l)
        x = _rms(h, gain("norm2", l), cfg.rms_eps)
        h = h + mat(torch.nn.functional.silu(mat(x, "wg", l)) * mat(x, "wu", l), "wd", l)
    rows = torch.cat([torch.arange(s[0] + s[1], s[0] + s[1] + s[2], device=dev) for s in seqs])
    return mat(_rms(h[rows], gain("norm_f"), cfg.rms_eps), "lm_head", -1).cpu()
