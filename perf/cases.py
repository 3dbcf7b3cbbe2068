"""Workloads of the decoding path: what a program that decodes with this framework calls, at the sizes it calls it with.

Four kinds of pass:
  verify   one pass of the target over the rows of a speculation (a chain of drafted tokens, a token tree, or the single row of
           plain decoding) on top of a committed context: logits of every row, their logsumexps, the drafted tokens' likelihoods
  prefill  a prompt through the model in causal chunks: the keys and values it leaves in the cache
  draft    one beam step of the draft model
  decide   what is decided on given logits: warped distributions, the beam's survivors, the tree, acceptance, the next token

Models are decoders with random weights of the widths the framework's workloads use, most of them with a few of their layers
(a layer's cost does not depend on how many follow); one verify case is a whole model.  Every input is made from the seed.
"""
import ctypes
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2407_09722_amd import binding as mb
from paper_2407_09722_amd.engine import Engine

EPS, THETA = 1e-5, 10000.0
PAGE = 16


# ---- the cases -------------------------------------------------------------------------------------------------------

def _widths(d, heads, kv_heads, head_dim, ffn, vocab, dtype="bf16"):
    return dict(d=d, heads=heads, kv_heads=kv_heads, head_dim=head_dim, ffn=ffn, vocab=vocab, dtype=dtype)


TINY = _widths(256, 4, 4, 64, 688, 1024, "fp32")
SMALL = _widths(768, 12, 12, 64, 2048, 32000)
W7B = _widths(4096, 32, 32, 128, 11008, 32000)
W13B = _widths(5120, 40, 40, 128, 13824, 32000)
DRAFT_S = _widths(768, 12, 12, 64, 3072, 32000)
DRAFT_L = _widths(2048, 32, 4, 64, 5632, 32000)


def _case(name, do, widths, layers, batch, gamma, beam, mode, context, **more):
    return dict(name=name, do=do, layers=layers, **widths, batch=batch, gamma=gamma, beam=beam, mode=mode, context=context, **more)


def listed():
    return [
        # the smallest: a toy pair in float32, whole, a chain of four tokens: latency and launches
        _case("verify_tiny_f32", "verify", TINY, 4, 1, 4, 2, "chain", 77),
        # plain decoding, one token of one sequence, of a small bfloat16 model, whole: launches again
        _case("decode_small", "verify", SMALL, 12, 1, 4, 4, "one", 255),
        # the headline: a whole 7B-shaped target verifies a chain of four drafted tokens after a 512-token prompt
        _case("verify_7b_whole", "verify", W7B, 32, 1, 4, 4, "chain", 511),
        # layers of the same target on a tree of 4 beams x 4 levels (17 rows), 2048-token context
        _case("tree_7b", "verify", W7B, 4, 1, 4, 4, "tree", 2047),
        # eight requests decoded together, chains of four, contexts of different lengths (40 rows)
        _case("batch_7b", "verify", W7B, 4, 8, 4, 4, "chain", 701),
        # layers of a 13B-shaped target: four requests, trees of 8 beams x 5 levels (164 rows), 4096-token contexts
        _case("tree_13b", "verify", W13B, 4, 4, 5, 8, "tree", 4095),
        # the prompt of a long request on the 7B-shaped target
        _case("prefill_7b", "prefill", W7B, 4, 1, 4, 4, "chain", 2047),
        # four ragged-length prompts of a batch on the 13B-shaped target
        _case("prefill_13b", "prefill", W13B, 4, 4, 5, 8, "tree", 509),
        # the same prompts' share of the draft model: grouped-query heads, whole
        _case("prefill_draft", "prefill", DRAFT_L, 22, 4, 5, 8, "tree", 1023),
        # a beam step of the 7B pair's two-layer draft: the many small launches of the draft phase
        _case("draft_small", "draft", DRAFT_S, 2, 1, 4, 4, "chain", 513, step=2),
        # a beam step of the 13B pair's draft, whole: 4 requests x 8 beams over 4096-token contexts, grouped-query heads
        _case("draft_large", "draft", DRAFT_L, 22, 4, 5, 8, "tree", 4099, step=3),
        # the decisions of an iteration in the warped, sampled setting
        _case("decide_warped", "decide", DRAFT_S, 1, 4, 4, 4, "tree", 600),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["verify", "verify", "verify", "prefill", "prefill", "draft", "decide"])
    while True:
        head_dim = rng.choice([64, 128])
        heads = _log(rng, 2, 40 if head_dim == 128 else 32)
        kv_heads = heads // rng.choice([g for g in (1, 1, 2, 4, 8) if heads % g == 0])
        d = heads * head_dim
        dtype = "fp32" if d <= 512 and rng.random() < 0.5 else "bf16"
        widths = _widths(d, heads, kv_heads, head_dim, max(64, int(d * rng.uniform(2.5, 4.0)) // 32 * 32),
                         rng.choice([32000, 16 * _log(rng, 64, 2000)]), dtype)
        layers = rng.randint(1, 4)
        batch = _log(rng, 1, 16 if do == "verify" else 4)
        gamma, beam = rng.randint(1, 8), rng.randint(1, 8)
        mode = rng.choice(["chain", "tree", "one"] if do == "verify" else ["chain", "tree"])
        rows = {"chain": 1 + gamma, "tree": 1 + gamma * beam, "one": 1}[mode]
        if rows > 64 or gamma + 1 + (gamma - 1) * beam > 64 or batch * max(rows, 1 + gamma, beam) > 256:
            continue
        context = _log(rng, 16, 4096 if do in ("verify", "draft") else 2048)
        if do == "prefill" and (dtype == "fp32" and context > 256 or batch * context > 4096):
            continue
        more = dict(step=rng.randrange(gamma)) if do == "draft" else {}
        c = _case("", do, widths, layers, batch, gamma, beam, mode, context, **more)
        del c["name"]
        return c


# ---- inputs ----------------------------------------------------------------------------------------------------------

def _generator(seed, *key):
    n = seed & 0xFFFFFFFF
    for k in key:
        n = (n * 1000003 + k + 1) % (1 << 61)
    return torch.Generator(device="cuda").manual_seed(n)


def _normal(shape, std, dtype, seed, *key, mean=0.0):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(mean, std, generator=_generator(seed, *key))


def _integers(hi, shape, seed, *key):
    return torch.randint(0, hi, shape, dtype=torch.int32, device="cuda", generator=_generator(seed, *key))


KINDS = ("embed", "g_attn", "w_qkv", "w_o", "g_ffn", "w_gu", "w_d", "g_final", "unembed")


def _weight(c, seed, kind, layer=0):
    """One weight tensor, row-major [out_features][in_features]: std 0.02 as a trained decoder's, logits of std 3."""
    d, f, V, hhd = c["d"], c["ffn"], c["vocab"], c["heads"] * c["head_dim"]
    shape = {"embed": (V, d), "unembed": (V, d), "w_qkv": (hhd + 2 * c["kv_heads"] * c["head_dim"], d), "w_o": (d, hhd), "w_gu": (2 * f, d),
             "w_d": (d, f)}.get(kind, (d,))
    key = (1, KINDS.index(kind), layer)
    if kind.startswith("g_"):
        return _normal(shape, 0.1, torch.float32, seed, *key, mean=1.0)
    std = 3.0 / math.sqrt(d) if kind == "unembed" else 0.02
    return _normal(shape, std, torch.float32 if c["dtype"] == "fp32" else torch.bfloat16, seed, *key)


class _Model:
    """Weights on the GPU in the layout the kernels stream, and the descriptor that points at them."""

    def __init__(self, c, seed):
        self.shape = SimpleNamespace(n_layers=c["layers"], d_model=c["d"], n_heads=c["heads"], n_kv_heads=c["kv_heads"], head_dim=c["head_dim"],
                                     d_ffn=c["ffn"], vocab=c["vocab"], dtype=c["dtype"])
        names = [("embed", 0)] + [(k, l) for l in range(c["layers"]) for k in KINDS[1:7]] + [("g_final", 0), ("unembed", 0)]
        self.tensors = []
        for kind, layer in names:
            w = _weight(c, seed, kind, layer)
            if w.dtype == torch.bfloat16 and kind != "embed":
                packed = torch.empty_like(w)
                mode = {"w_qkv": mb.MTAD_PACK_QKV, "w_gu": mb.MTAD_PACK_GATE_UP}.get(kind, mb.MTAD_PACK_PLAIN)
                mb.mtad_pack_matrix(mode, w, packed, w.shape[0], w.shape[1], c["head_dim"])
                w = packed
            self.tensors.append(w)
        self._ptrs = (ctypes.c_void_p * len(self.tensors))(*[t.data_ptr() for t in self.tensors])
        s = self.shape
        self.desc = mb.mtad_model(s.n_layers, s.d_model, s.n_heads, s.n_kv_heads, s.head_dim, s.d_ffn, s.vocab, 1 if s.dtype == "bf16" else 0,
                                  EPS, THETA, ctypes.cast(self._ptrs, ctypes.POINTER(ctypes.c_void_p)))


def _rows(c):
    return {"chain": 1 + c["gamma"], "tree": 1 + c["gamma"] * c["beam"], "one": 1}[c["mode"]]


def _lens(c, seed):
    """Committed tokens of each sequence: the requests of a batch differ by some tens of tokens."""
    r = np.random.default_rng([seed & 0xFFFFFFFF, 7])
    spread = min(64, c["context"] // 4)
    return [c["context"] - (int(r.integers(0, spread + 1)) if s else 0) for s in range(c["batch"])]


def _max_context(c):
    return c["context"] + 64 + 64


def _pages(c, seed):
    max_pages = -(-_max_context(c) // PAGE)
    perm = np.random.default_rng([seed & 0xFFFFFFFF, 8]).permutation(max_pages * c["batch"]).astype(np.int32)
    return perm.reshape(c["batch"], max_pages)


def _cache(c, seed, which):
    """Keys (which 0) or values (1) of a context that lies in the cache: the spread that std 0.02 weights give normalised rows."""
    n_pages = c["batch"] * -(-_max_context(c) // PAGE)
    return _normal((c["layers"], n_pages, PAGE, c["kv_heads"], c["head_dim"]), 0.02 * math.sqrt(c["d"]),
                   torch.float32 if c["dtype"] == "fp32" else torch.float16, seed, 2, which)


def _tree(c, seed):
    """Rows of a speculation: token, parent row, depth, beam of every row, and the rows each row sees."""
    r = np.random.default_rng([seed & 0xFFFFFFFF, 9])
    B, M, g, b = c["batch"], _rows(c), c["gamma"], c["beam"]
    tok = r.integers(0, c["vocab"], (B, M)).astype(np.int32)
    parent, depth, src = np.full((B, M), -1, np.int32), np.zeros((B, M), np.int32), np.full((B, M), -1, np.int32)
    sees = np.zeros((B, M, M), bool)
    for s in range(B):
        sees[s, 0, 0] = True
        for row in range(1, M):
            i, k = (row - 1, 0) if c["mode"] == "chain" else divmod(row - 1, b)
            p = i if c["mode"] == "chain" else 0 if i == 0 else 1 + (i - 1) * b + int(r.integers(0, b))
            parent[s, row], depth[s, row], src[s, row] = p, i + 1, k
            sees[s, row] = sees[s, p]
            sees[s, row, row] = True
    qref = -np.cumsum(r.uniform(2.0, 4.0, (B, g)), 1).astype(np.float32)
    return SimpleNamespace(tok=tok, parent=parent, depth=depth, src=src, sees=sees, qref=qref)


def _beams(c, seed):
    """A beam history and the catch-up tokens before it: survivors of every step, best first."""
    r = np.random.default_rng([seed & 0xFFFFFFFF, 10])
    B, g, b = c["batch"], c["gamma"], c["beam"]
    tok = r.integers(0, c["vocab"], (B, g, b)).astype(np.int32)
    parent = r.integers(0, b, (B, g, b)).astype(np.int32)
    parent[:, 0] = 0
    cum = np.sort(-3.0 * np.arange(1, g + 1)[None, :, None] - r.uniform(0, 4, (B, g, b)), axis=2)[:, :, ::-1].astype(np.float32)
    cnt = r.integers(1, 3, B).astype(np.int32) if g > 0 else np.ones(B, np.int32)
    catchup = r.integers(0, c["vocab"], (B, g + 1)).astype(np.int32)
    return SimpleNamespace(tok=tok, parent=parent, cum=np.ascontiguousarray(cum), cnt=cnt, catchup=catchup)


def _gpu(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _engine(c, model, other, seed, drafting):
    mode = "mmtad" if c["mode"] == "tree" else "mtad"
    target, draft = (other, model) if drafting else (model, other)
    return Engine(target, draft, batch=c["batch"], gamma=c["gamma"], beam=c["beam"], mode=mode, max_context=_max_context(c),
                  prefill_rows=min(64, 256 // c["batch"]), page_size=PAGE)


def prepare(case, seed):
    c = case
    other = _Model(dict(layers=1, **_widths(128, 2, 2, 64, 256, c["vocab"], c["dtype"])), seed)
    model = _Model(c, seed)
    eng = _engine(c, model, other, seed, c["do"] == "draft")
    st = SimpleNamespace(case=c, eng=eng, model=model, other=other, seed=seed)
    kv = eng.dkv if c["do"] == "draft" else eng.tkv
    kv.page_table.copy_(_gpu(_pages(c, seed)))
    B, M, V = c["batch"], _rows(c), c["vocab"]
    if c["do"] == "prefill":
        st.tokens = _integers(V, (B, c["context"]), seed, 3)
        return st
    kv.k.copy_(_cache(c, seed, 0))
    kv.v.copy_(_cache(c, seed, 1))
    kv.len.copy_(_gpu(np.asarray(_lens(c, seed), np.int32)))
    if c["do"] == "draft":
        h = _beams(c, seed)
        eng.h_tok.copy_(_gpu(h.tok)), eng.h_parent.copy_(_gpu(h.parent)), eng.h_cum.copy_(_gpu(h.cum))
        eng.catchup_tok.copy_(_gpu(h.catchup)), eng.catchup_cnt.copy_(_gpu(h.cnt))
        return st
    st.logits, st.row_lse, st.logp_cond = (torch.zeros(s, device="cuda") for s in ((B, M, V), (B, M), (B, M)))
    t = _tree(c, seed)
    eng.root_tok.copy_(_gpu(t.tok[:, 0]))
    if c["mode"] == "one":
        st.tree = eng.ar_tree
        return st
    st.tree = eng.tree
    for to, x in ((eng.t_tok, t.tok), (eng.t_parent, t.parent), (eng.t_depth, t.depth), (eng.t_src, t.src), (eng.t_qref, t.qref)):
        to.copy_(_gpu(x))
    eng.t_mask.copy_(_gpu((t.sees.astype(np.uint64) << np.arange(M, dtype=np.uint64)).sum(2).astype(np.int64)))
    if c["do"] == "decide":
        h = _beams(c, seed)
        eng.h_tok.copy_(_gpu(h.tok)), eng.h_parent.copy_(_gpu(h.parent)), eng.h_cum.copy_(_gpu(h.cum)), eng.catchup_cnt.copy_(_gpu(h.cnt))
        st.rows = max(c["beam"], c["gamma"] + 1 if c["gamma"] == 1 else 0)
        st.draft_rows = _normal((B, st.rows, V), 3.0, torch.float32, seed, 4)
        st.target_rows = _normal((B, M, V), 3.0, torch.float32, seed, 5)
        st.draft_work, st.draft_lse = torch.empty_like(st.draft_rows), torch.zeros(B, st.rows, device="cuda")
        st.logp_cond = _normal((B, M), 1.5, torch.float32, seed, 6, mean=-3.0)
        st.tau = 0.1
    return st


# ---- one pass --------------------------------------------------------------------------------------------------------

def run(st):
    c, eng = st.case, st.eng
    if c["do"] == "verify":
        mb.mtad_verify_tree(eng.ctx, st.model.desc, eng.tkv.desc, eng.root_tok, st.tree, st.logp_cond, st.row_lse, st.logits)
        return {"logits": st.logits, "row_lse": st.row_lse, "logp_cond": st.logp_cond}
    if c["do"] == "prefill":
        eng.tkv.len.zero_()
        mb.mtad_prefill(eng.ctx, st.model.desc, eng.tkv.desc, st.tokens, c["context"])
        return {"k": eng.tkv.k, "v": eng.tkv.v, "len": eng.tkv.len}
    if c["do"] == "draft":
        # The survivors' likelihoods say which candidates were kept.  Their token ids are not compared: with random weights two
        # candidates often lie within the rounding of a 16-bit model and may trade places ("decide" compares ids).
        mb.mtad_draft_beam_step(eng.ctx, st.model.desc, eng.dkv.desc, eng.hist, c["step"], eng.state)
        return {"cum_logq": eng.h_cum}
    B, M, V, gamma = c["batch"], _rows(c), c["vocab"], c["gamma"]
    st.draft_work.copy_(st.draft_rows)  # the logits a pass would have left: warping works in place
    mb.mtad_k_warp_rows(st.draft_work, st.draft_lse, B * st.rows, V, 10, 0.9)
    mb.mtad_k_beam_topb(eng.ctx, st.draft_work, st.draft_lse, eng.hist, gamma - 1, eng.catchup_cnt, eng.dkv.len, st.rows, V, 1, st.seed & 0xFFFF)
    mb.mtad_build_tree(eng.ctx, eng.hist, eng.mode, eng.tree)
    st.logits.copy_(st.target_rows)
    mb.mtad_k_warp_rows(st.logits, st.row_lse, B * M, V, 10, 0.9)
    mb.mtad_accept(eng.ctx, eng.tree, st.logp_cond, st.logits, V, eng.tkv.desc, st.tau, eng.mode, 1, st.seed & 0xFFFF, eng.acc)
    return {"draft": st.draft_work, "target": st.logits, "cum_logq": eng.h_cum, "survivors": [eng.h_tok, eng.h_parent],
            "tree": [eng.t_tok, eng.t_parent, eng.t_depth, eng.t_src, eng.t_mask], "qref": eng.t_qref,
            "accepted": [eng.eta, eng.path, eng.bonus_row, eng.bonus_tok, eng.out_tok, eng.out_cnt]}


# ---- what a pass cannot do without -----------------------------------------------------------------------------------

def work(case):
    c = case
    d, f, V, hd, H, KVH, L, B = c["d"], c["ffn"], c["vocab"], c["head_dim"], c["heads"], c["kv_heads"], c["layers"], c["batch"]
    e = 4 if c["dtype"] == "fp32" else 2
    if c["do"] == "decide":
        n = B * (max(c["beam"], c["gamma"] + 1 if c["gamma"] == 1 else 0) + _rows(c)) * V
        return {"bytes": 2 * 4 * n, "flops": 4 * n}
    layer = d * (H + 2 * KVH) * hd + d * H * hd + 3 * d * f
    if c["do"] == "prefill":  # the last layer's part of the cache needs its keys and values only
        n = c["context"]
        weights = (L - 1) * layer + 2 * d * KVH * hd
        return {"bytes": e * (weights + B * n * d + 2 * L * B * n * KVH * hd),
                "flops": 2 * B * n * weights + (L - 1) * B * 4 * H * hd * n * (n + 1) // 2}
    rows = B * (_rows(c) if c["do"] == "verify" else 1 if c["step"] == 0 else c["beam"])
    weights = L * layer + V * d
    seen = c["context"] + rows // B
    out = 4 * rows * (V + 2) if c["do"] == "verify" else 12 * B * c["beam"]
    return {"bytes": e * (weights + rows * d + 2 * L * KVH * hd * (B * c["context"] + rows)) + out,
            "flops": 2 * rows * weights + L * 4 * rows * seen * H * hd}


def tolerance(case):
    """About four times the distance from the 64-bit results that was measured over the listed cases and drawn ones."""
    if case["do"] == "decide":
        return {"rel": 5e-7}  # measured 7e-8
    if case["dtype"] == "fp32":
        return {"rel": 4e-6}  # 3e-7 at four layers, more in the keys of long prompts
    if case["do"] == "prefill":
        return {"rel": 3e-3}  # 7e-4: a half-precision cache, from four layers on
    if case["do"] == "draft":
        return {"rel": 4e-5}  # 1e-6 to 5e-6, and candidates within that may trade places
    return {"rel": 8e-4 if case["layers"] > 12 else 4e-4}  # 1.7e-4 for 32 layers, 3e-5 to 1e-4 for 1 to 12


# ---- the same in 64 bits ---------------------------------------------------------------------------------------------

def _rms(h, g):
    return h / torch.sqrt((h * h).mean(1, keepdim=True) + EPS) * g


def _layer(c, seed, l, h, angle, attend):
    """One decoder layer over all rows; attend(q, k, v) gives the attention output.  Returns (h, k, v)."""
    hd, H, KVH, f = c["head_dim"], c["heads"], c["kv_heads"], c["ffn"]
    w = lambda kind: _weight(c, seed, kind, l).double()  # noqa: E731
    qkv = (_rms(h, w("g_attn")) @ w("w_qkv").T).view(h.shape[0], H + 2 * KVH, hd)
    q, k, v = qkv[:, :H], qkv[:, H:H + KVH], qkv[:, H + KVH:]
    cos, sin = angle.cos()[:, None], angle.sin()[:, None]
    turn = lambda x: torch.cat([x[..., :hd // 2] * cos - x[..., hd // 2:] * sin, x[..., hd // 2:] * cos + x[..., :hd // 2] * sin], -1)  # noqa: E731
    q, k = turn(q), turn(k)
    h = h + attend(q, k, v).reshape(h.shape[0], H * hd) @ w("w_o").T
    gu = _rms(h, w("g_ffn")) @ w("w_gu").T
    return h + (torch.nn.functional.silu(gu[:, :f]) * gu[:, f:]) @ w("w_d").T, k, v


def _angles(c, pos):
    half = c["head_dim"] // 2
    return pos.double()[:, None] * torch.pow(torch.tensor(THETA, dtype=torch.float64, device="cuda"),
                                             -torch.arange(half, dtype=torch.float64, device="cuda") / half)


def _softmax_out(c, q, k, v, sees):
    """q [n, H, hd] over k, v [m, KVH, hd]; sees [n, m]."""
    g = c["heads"] // c["kv_heads"]
    k, v = k.repeat_interleave(g, 1).permute(1, 2, 0).contiguous(), v.repeat_interleave(g, 1).permute(1, 0, 2).contiguous()
    s = torch.matmul(q.permute(1, 0, 2).contiguous(), k) / math.sqrt(c["head_dim"])
    return torch.matmul(s.masked_fill_(~sees, -math.inf).softmax(-1), v).permute(1, 0, 2)


def _head(c, seed, h):
    return _rms(h, _weight(c, seed, "g_final").double()) @ _weight(c, seed, "unembed").double().T


def _speculate(c, seed, tok, pos, sees, extra):
    """Rows tok [B][M] at positions pos over the committed context, `extra` [B] more cached tokens and each other (sees [B][M][extra + M])."""
    B, M = tok.shape
    lens, pages = _lens(c, seed), torch.from_numpy(_pages(c, seed)).long().cuda()
    caches = [_cache(c, seed, i) for i in (0, 1)]
    h = _weight(c, seed, "embed")[tok.reshape(-1).long()].double()
    angle = _angles(c, pos.reshape(-1))
    for l in range(c["layers"]):
        def attend(q, k, v):
            out = []
            for s in range(B):
                t = torch.arange(lens[s] + extra[s], device="cuda")
                at = pages[s, t // PAGE] * PAGE + t % PAGE
                old = [x[l].reshape(-1, c["kv_heads"], c["head_dim"])[at].double() for x in caches]
                rows = slice(s * M, (s + 1) * M)
                see = torch.cat([torch.ones(M, lens[s], dtype=torch.bool, device="cuda"), sees[s]], 1)
                out.append(_softmax_out(c, q[rows], torch.cat([old[0], k[rows]]), torch.cat([old[1], v[rows]]), see))
            return torch.cat(out)
        h = _layer(c, seed, l, h, angle, attend)[0]
    return _head(c, seed, h).view(B, M, -1)


def _warped(rows):
    """log of the warped distribution: the 10 most likely tokens, of those the shortest prefix with more than 0.9 of their sum."""
    x = rows.double()
    top, at = x.topk(10, -1)
    p = top.softmax(-1)
    kept = torch.cat([torch.zeros_like(p[..., :1]), p.cumsum(-1)[..., :-1]], -1) <= 0.9
    p = torch.where(kept, p, torch.zeros_like(p))
    return torch.full_like(x, -math.inf).scatter_(-1, at, (p / p.sum(-1, keepdim=True)).log())


def exact(case, seed):
    c = case
    B, M = c["batch"], _rows(c)
    if c["do"] == "decide":
        rows = max(c["beam"], c["gamma"] + 1 if c["gamma"] == 1 else 0)
        return {"draft": _warped(_normal((B, rows, c["vocab"]), 3.0, torch.float32, seed, 4)),
                "target": _warped(_normal((B, M, c["vocab"]), 3.0, torch.float32, seed, 5)), "cum_logq": None, "survivors": None, "tree": None,
                "qref": None, "accepted": None}
    if c["do"] == "prefill":
        n = c["context"]
        tokens = _integers(c["vocab"], (B, n), seed, 3)
        pages = torch.from_numpy(_pages(c, seed)).long().cuda()
        t = torch.arange(n, device="cuda")
        at = [pages[s, t // PAGE] * PAGE + t % PAGE for s in range(B)]
        causal = torch.ones(n, n, dtype=torch.bool, device="cuda").tril()
        h = _weight(c, seed, "embed")[tokens.reshape(-1).long()].double()
        angle = _angles(c, t.repeat(B))
        got = [torch.zeros(c["layers"], B * pages.shape[1] * PAGE, c["kv_heads"], c["head_dim"], dtype=torch.float64, device="cuda") for _ in range(2)]

        def attend(q, k, v):
            return torch.cat([_softmax_out(c, q[s * n:(s + 1) * n], k[s * n:(s + 1) * n], v[s * n:(s + 1) * n], causal) for s in range(B)])
        for l in range(c["layers"]):
            h, k, v = _layer(c, seed, l, h, angle, attend)
            for s in range(B):
                got[0][l, at[s]], got[1][l, at[s]] = k[s * n:(s + 1) * n], v[s * n:(s + 1) * n]
        shape = (c["layers"], B * pages.shape[1], PAGE, c["kv_heads"], c["head_dim"])
        return {"k": got[0].view(shape), "v": got[1].view(shape), "len": None}
    lens = torch.tensor(_lens(c, seed), device="cuda")[:, None]
    if c["do"] == "verify":
        t = _tree(c, seed)
        logits = _speculate(c, seed, _gpu(t.tok), lens + _gpu(t.depth), _gpu(t.sees), [0] * B)
        lse = torch.logsumexp(logits, -1)
        parent = _gpu(t.parent).long().clamp(min=0)
        cond = logits.gather(1, parent[..., None].expand(-1, -1, c["vocab"])).gather(2, _gpu(t.tok).long()[..., None])[..., 0] - lse.gather(1, parent)
        cond[:, 0] = 0
        return {"logits": logits, "row_lse": lse, "logp_cond": cond}
    h, step, b = _beams(c, seed), c["step"], c["beam"]
    cum = torch.from_numpy(h.cum).double()
    if step == 0:
        rows = int(h.cnt.max())
        tok, pos = _gpu(h.catchup[:, :rows]), lens + torch.arange(rows, device="cuda")
        sees = torch.ones(rows, rows, dtype=torch.bool, device="cuda").tril().expand(B, rows, rows)
        logits = _speculate(c, seed, tok, pos, sees, [0] * B)
        score = torch.stack([logits[s, int(h.cnt[s]) - 1].log_softmax(-1) for s in range(B)])
    else:
        extra = [int(h.cnt[s]) + (step - 1) * b for s in range(B)]
        sees = []
        for s in range(B):  # a beam sees the catch-up tokens, its ancestors and itself
            cnt, see = int(h.cnt[s]), torch.zeros(b, extra[s] + b, dtype=torch.bool)
            see[:, :cnt] = True
            for r in range(b):
                see[r, extra[s] + r] = True
                j = r
                for i in range(step - 1, 0, -1):
                    j = int(h.parent[s, i, j])
                    see[r, cnt + (i - 1) * b + j] = True
            sees.append(see.cuda())
        pos = lens + _gpu(h.cnt)[:, None] - 1 + step + torch.zeros(1, b, dtype=torch.int64, device="cuda")
        logits = _speculate(c, seed, _gpu(h.tok[:, step - 1]), pos, sees, extra)
        score = (logits.log_softmax(-1) + cum[:, step - 1].cuda()[..., None]).reshape(B, -1)
    cum[:, step] = score.topk(b, -1)[0].cpu()
    return {"cum_logq": cum}
