"""The work a program gives this library, as timed cases: draft steps (greedy and
sampled, with and without context rows to append), the teacher-forced training
forward, the target's verify pass with acceptance and cache commit, and the two
acceptance rules on their own.

`listed()` and `draw()` give cases, `prepare()` the buffers and the model handle
a program holds before a call, `run()` one pass through the entry points of the
binding, `exact()` the same outputs in 64 bits from plain torch.  Values follow
the library's own synthetic recipe: matrices and GRU biases N(0, 0.02), unit
norm gains, N(0, 1) context keys, values and hidden states.
"""
import math
from types import SimpleNamespace

import torch

from paper_2605_29707_amd import binding as bd

BLOCK = 16


def _dims(hidden, layers, nq, ffn, *, nkv=8, head_dim=128, vocab=151936, dtype="bf16", fuse=5):
    return dict(hidden=hidden, n_layers=layers, n_q_heads=nq, n_kv_heads=nkv, head_dim=head_dim, ffn=ffn,
                vocab=vocab, block=BLOCK, gru_hidden=1024, rank=256, mask_id=vocab - 1, rms_eps=1e-6,
                rope_theta=1e6, dtype=dtype, ctx_fuse_layers=fuse)


MODELS = {
    "tiny": _dims(256, 2, 4, 1024, nkv=2, head_dim=64, vocab=4096, dtype="f32", fuse=0),
    "4b": _dims(2560, 5, 32, 9728),
    "8b": _dims(4096, 5, 32, 12288),
    "32b": _dims(5120, 5, 64, 25600),
    "8b_target": _dims(4096, 36, 32, 12288, fuse=0),
}


def listed():
    return [
        # the smallest call: a tiny fp32 drafter, its whole context projected from hidden states; launches count
        dict(name="draft_tiny_f32", kind="draft", model="tiny", batch=1, ctx=128, branch=1, n_new=128, ragged=False),
        # one interactive user: the latency of a greedy step and its chain
        dict(name="draft_8b_bs1", kind="draft", model="8b", batch=1, ctx=1024, branch=1, n_new=0, ragged=False),
        # the same user at temperature 1, the tokens of the last cycle appended first
        dict(name="sample_8b_bs1_append", kind="sampled", model="8b", batch=1, ctx=1531, n_new=5, ragged=False,
             temperature=1.0),
        # a few users of a small model with long contexts
        dict(name="draft_4b_bs4_ctx8k", kind="draft", model="4b", batch=4, ctx=8192, branch=1, n_new=0, ragged=False),
        # a few users at different lengths, two candidates a depth; an odd batch
        dict(name="draft_8b_bs7_ragged", kind="draft", model="8b", batch=7, ctx=1777, branch=2, n_new=0, ragged=True),
        # serving: a full batch with a tree of four candidates a depth
        dict(name="draft_8b_bs32_b4", kind="draft", model="8b", batch=32, ctx=2048, branch=4, n_new=0, ragged=False),
        # serving a large model
        dict(name="draft_32b_bs16", kind="draft", model="32b", batch=16, ctx=4096, branch=1, n_new=0, ragged=False),
        # the forward and loss of a training batch, ragged contexts
        dict(name="train_8b_bs16", kind="train", model="8b", batch=16, ctx=512, ragged=True),
        # the target's pass over a drafted chain, acceptance and commit: the other half of every cycle
        dict(name="verify_8b_chain", kind="verify", model="8b_target", batch=1, ctx=1024, branch=1, ragged=False,
             logits="f32"),
        # the same for four users with trees of two candidates a depth
        dict(name="verify_8b_bs4_tree", kind="verify", model="8b_target", batch=4, ctx=1500, branch=2, ragged=True,
             logits="bf16"),
        # greedy acceptance of a full serving batch of trees
        dict(name="accept_bs32_b4", kind="accept", batch=32, branch=4, vocab=151936, logits="bf16"),
        # acceptance by the sampling rule
        dict(name="accept_sampled_bs8", kind="accept_sampled", batch=8, vocab=151936, logits="bf16", temperature=0.8),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["draft"] * 4 + ["sampled", "train", "verify", "accept", "accept_sampled"])
    if kind == "draft":
        model = rng.choice(["8b", "8b", "4b", "32b", "tiny"])
        batch = _log_int(rng, 1, {"32b": 16, "tiny": 8}.get(model, 32))
        ctx = _log_int(rng, 64, min(8192, 65536 // batch)) if model != "tiny" else _log_int(rng, 32, 512)
        n_new = ctx if model == "tiny" else rng.choice([0, 0, rng.randint(1, BLOCK)])
        return dict(kind=kind, model=model, batch=batch, ctx=ctx, branch=rng.choice([1, 1, 2, 4]), n_new=n_new,
                    ragged=model != "tiny" and rng.random() < 0.7)
    if kind == "sampled":
        batch = _log_int(rng, 1, 16)
        return dict(kind=kind, model=rng.choice(["8b", "4b"]), batch=batch, ctx=_log_int(rng, 64, 4096),
                    n_new=rng.choice([0, rng.randint(1, BLOCK)]), ragged=rng.random() < 0.7,
                    temperature=rng.choice([0.6, 0.8, 1.0]))
    if kind == "train":
        return dict(kind=kind, model=rng.choice(["8b", "4b"]), batch=_log_int(rng, 1, 16),
                    ctx=_log_int(rng, 64, 2048), ragged=True)
    if kind == "verify":
        return dict(kind=kind, model="8b_target", batch=rng.randint(1, 4), ctx=_log_int(rng, 64, 1500),
                    branch=rng.choice([1, 2]), ragged=True, logits=rng.choice(["bf16", "f32"]))
    vocab = rng.choice([32000, 50257, 128256, 151936])
    if kind == "accept":
        return dict(kind=kind, batch=_log_int(rng, 1, 32), branch=rng.choice([1, 2, 4]), vocab=vocab,
                    logits=rng.choice(["bf16", "f32"]))
    return dict(kind=kind, batch=_log_int(rng, 1, 16), vocab=vocab, logits=rng.choice(["bf16", "f32"]),
                temperature=rng.choice([0.6, 0.8, 1.0]))


# --------------------------------------------------------------------------
# inputs, from the seed alone
# --------------------------------------------------------------------------
DEV = "cuda"
_LAYER = ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down")
_BORROWED = ("embed", "final_norm", "gru_b_ih", "gru_b_hh")


def _cfg(case):
    return SimpleNamespace(**MODELS[case["model"]])


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 4099 + stream)
    return g


def _dtype(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _cap(case, cfg):
    """Cache capacity: room for the next block, in steps a program would allocate."""
    step = 1024 if cfg.head_dim == 128 else 128
    return -(-(case["ctx"] + 2 * BLOCK) // step) * step


def _weights(cfg, seed, head=True):
    g, dt = _gen(seed, 1), _dtype(cfg.dtype)
    d, ds, r, V = cfg.hidden, cfg.gru_hidden, cfg.rank, cfg.vocab
    qd, kvd = cfg.n_q_heads * cfg.head_dim, cfg.n_kv_heads * cfg.head_dim

    def mat(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=dt).mul_(0.02)

    def ones(n):
        return torch.ones(n, device=DEV, dtype=dt)

    shapes = dict(wq=(qd, d), wk=(kvd, d), wv=(kvd, d), wo=(d, qd), w_gate=(cfg.ffn, d), w_up=(cfg.ffn, d),
                  w_down=(d, cfg.ffn))
    w = {"embed": mat(V, d), "lm_head": mat(V, d), "final_norm": ones(d), "layers": []}
    for _ in range(cfg.n_layers):
        lw = {k: mat(*shapes[k]) for k in _LAYER}
        lw.update(attn_norm=ones(d), ffn_norm=ones(d), q_norm=ones(cfg.head_dim), k_norm=ones(cfg.head_dim))
        w["layers"].append(lw)
    if head:
        w.update(gru_w_ih=mat(3 * ds, d), gru_w_hh=mat(3 * ds, ds), gru_b_ih=mat(3 * ds), gru_b_hh=mat(3 * ds),
                 w1=mat(r, d + ds), w2=mat(V, r))
        if cfg.ctx_fuse_layers:
            w["ctx_fc"] = mat(d, cfg.ctx_fuse_layers * d)
    return w


def _model(cfg, seed, head=True):
    w = _weights(cfg, seed, head)
    m = bd.DominoModel(cfg, w, target=not head)
    # the handle has its own copies; only these stay borrowed
    for k in [k for k in w if k != "layers" and k not in _BORROWED]:
        del w[k]
    for lw in w["layers"]:
        for k in _LAYER:
            del lw[k]
    return m


def _lens(case, seed):
    n = torch.full((case["batch"],), case["ctx"], dtype=torch.int32, device=DEV)
    if case["ragged"] and case["batch"] > 1:
        lo = max(case.get("n_new", 0), case["ctx"] // 4)
        n[:-1] = torch.randint(lo, case["ctx"] + 1, (case["batch"] - 1,), generator=_gen(seed, 2), device=DEV,
                               dtype=torch.int32)
    return n


def _context(case, cfg, seed):
    """Anchors, lengths, the K/V caches and the hidden rows to append."""
    g, b, cap = _gen(seed, 3), case["batch"], _cap(case, cfg)
    s = dict(anchor=torch.randint(0, cfg.vocab - 1, (b,), generator=g, device=DEV, dtype=torch.int32),
             lens=_lens(case, seed), cap=cap)
    shape = (cfg.n_layers, b, cap, cfg.n_kv_heads, cfg.head_dim)
    s["ck"] = torch.randn(shape, generator=g, device=DEV, dtype=_dtype(cfg.dtype))
    s["cv"] = torch.randn(shape, generator=g, device=DEV, dtype=_dtype(cfg.dtype))
    n = case.get("n_new", 0)
    s["new"] = None
    if n:
        width = cfg.hidden * max(1, cfg.ctx_fuse_layers)
        s["new"] = torch.randn((b, n, width), generator=g, device=DEV)
    return s


def _i32(*shape):
    return torch.empty(shape, dtype=torch.int32, device=DEV)


def _tree_buffers(batch, nodes):
    return [_i32(batch, nodes) for _ in range(4)] + [torch.empty((batch, nodes, nodes), dtype=torch.uint8, device=DEV)]


def _accept_buffers(batch):
    return dict(acc=_i32(batch), acc_nodes=_i32(batch, BLOCK - 1), out=_i32(batch, BLOCK))


def _random_tree(case, seed, vocab, anchor, lens):
    """A draft tree of random distinct tokens a depth, as the library lays it out."""
    g, b, beta = _gen(seed, 4), case["batch"], case.get("branch", 1)
    first = torch.randint(0, vocab - 8, (b, BLOCK - 1, 1), generator=g, device=DEV, dtype=torch.int32)
    top = (first + torch.arange(beta, device=DEV, dtype=torch.int32)).contiguous()
    tree = _tree_buffers(b, 1 + (BLOCK - 1) * beta)
    bd.domino_build_tree(top, anchor, lens, *tree[:4], ancestor_mask=tree[4])
    return tree


def prepare(case, seed):
    s, kind = dict(case=case), case["kind"]
    b = case["batch"]
    if kind in ("draft", "sampled", "train"):
        cfg = _cfg(case)
        beta, n = case.get("branch", 1), case.get("n_new", 0)
        s.update(_context(case, cfg, seed), model=_model(cfg, seed))
        s["hidden"] = torch.empty((b, BLOCK - 1, cfg.hidden), device=DEV)
        if kind == "train":
            s["labels"] = torch.randint(0, cfg.vocab, (b, BLOCK - 1), generator=_gen(seed, 5), device=DEV,
                                        dtype=torch.int32)
            s["loss"], s["ce"] = torch.empty(3, device=DEV), torch.empty((2, b, BLOCK - 1), device=DEV)
            nb = bd.domino_train_workspace_bytes(s["model"], b, s["cap"], 0)
        else:
            s["ids"], s["vals"] = _i32(b, BLOCK - 1, beta), torch.empty((b, BLOCK - 1, beta), device=DEV)
            s["tree"] = _tree_buffers(b, 1 + (BLOCK - 1) * beta)
            if kind == "sampled":
                s["final"] = torch.empty((b, BLOCK - 1, cfg.vocab), device=DEV)
                s["seed"] = case_seed(seed)
            nb = s["model"].workspace_bytes(b, s["cap"], n, beta)
        s["ws"] = torch.empty(nb, dtype=torch.uint8, device=DEV)
        return s
    s.update(_accept_buffers(b))
    if kind == "verify":
        cfg = _cfg(case)
        s.update(_context(case, cfg, seed), model=_model(cfg, seed, head=False))
        s["tree"] = _random_tree(case, seed, cfg.vocab, s["anchor"], s["lens"])
        nn = s["tree"][0].shape[1]
        s["logits"] = torch.empty((b, nn, cfg.vocab), device=DEV, dtype=_dtype(case["logits"]))
        s["new_lens"] = _i32(b)
        s["ws"] = torch.empty(bd.domino_target_workspace_bytes(s["model"], b, nn, s["cap"]), dtype=torch.uint8,
                              device=DEV)
        s["aws"] = torch.empty(bd.domino_verify_workspace_bytes(b, nn, cfg.vocab), dtype=torch.uint8, device=DEV)
        return s
    V, g = case["vocab"], _gen(seed, 6)
    anchor = torch.randint(0, V, (b,), generator=g, device=DEV, dtype=torch.int32)
    s["tree"] = _random_tree(case, seed, V, anchor, torch.full_like(anchor, 100))
    nn = s["tree"][0].shape[1]
    tok = s["tree"][0].long()
    if kind == "accept":
        lg = torch.randn((b, nn, V), generator=g, device=DEV, dtype=_dtype(case["logits"]))
        # the target agrees with a candidate of the next depth four times in five, mostly the first
        beta = case["branch"]
        for d in range(BLOCK - 1):
            node = 0 if d == 0 else 1 + (d - 1) * beta
            pick = (torch.rand(b, generator=g, device=DEV) ** 3 * beta).long() + 1 + d * beta
            hit = torch.rand(b, generator=g, device=DEV) < 0.8
            want = torch.where(hit, tok.gather(1, pick[:, None])[:, 0],
                               torch.randint(0, V, (b,), generator=g, device=DEV))
            lg[torch.arange(b, device=DEV), node, want] = 12.0
        s["logits"] = lg
        s["ws"] = torch.empty(bd.domino_verify_workspace_bytes(b, nn, V), dtype=torch.uint8, device=DEV)
        return s
    # sampling rule: drafts drawn from the draft distribution, a target close to it
    draft = torch.randn((b, BLOCK - 1, V), generator=g, device=DEV) * 2.5
    noise = torch.rand((b, BLOCK - 1, V), generator=g, device=DEV).clamp_(1e-7, 1 - 1e-7)
    drawn = (draft / case["temperature"] - noise.log().neg().log()).argmax(-1)
    tok[:, 1:] = drawn
    s["tree"][0].copy_(tok)
    lg = torch.randn((b, BLOCK, V), generator=g, device=DEV) * 0.3
    lg[:, :-1] += draft
    s["draft"], s["logits"], s["seed"] = draft, lg.to(_dtype(case["logits"])), case_seed(seed)
    s["ws"] = torch.empty(bd.domino_verify_sample_workspace_bytes(b, BLOCK, V), dtype=torch.uint8, device=DEV)
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("draft", "sampled"):
        kw = dict(ctx_hidden_new=s["new"], n_new=case["n_new"], debug={"hidden": s["hidden"]})
        out = {}
        if kind == "draft":
            bd.domino_draft_step(s["model"], s["anchor"], s["lens"], s["ck"], s["cv"], s["cap"], s["ids"], s["vals"],
                                 s["ws"], branch=case["branch"], **kw)
        else:
            bd.domino_draft_step_sampled(s["model"], s["anchor"], s["lens"], s["ck"], s["cv"], s["cap"], s["ids"],
                                         s["vals"], s["final"], s["ws"], case["temperature"], s["seed"], **kw)
            out["final_logits"] = s["final"]
        t = s["tree"]
        bd.domino_build_tree(s["ids"], s["anchor"], s["lens"], *t[:4], ancestor_mask=t[4])
        out.update(ids=s["ids"], vals=s["vals"], hidden=s["hidden"], tokens=t[0], parents=t[1], depths=t[2],
                   positions=t[3], mask=t[4])
        if case["n_new"]:
            out.update(ck=s["ck"], cv=s["cv"])
        return out
    if kind == "train":
        bd.domino_train_forward(s["model"], s["anchor"], s["lens"], s["ck"], s["cv"], s["cap"], s["labels"], 0.5, 15.0,
                                s["loss"], s["ws"], ce=s["ce"], debug={"hidden": s["hidden"]})
        return dict(loss=s["loss"], ce=s["ce"], hidden=s["hidden"])
    tok, par, _, pos, mask = s["tree"]
    done = dict(accept_len=s["acc"], accepted_nodes=s["acc_nodes"], out_tokens=s["out"])
    if kind == "verify":
        bd.domino_target_verify(s["model"], tok, pos, mask, s["lens"], s["ck"], s["cv"], s["cap"], s["logits"], s["ws"])
        bd.domino_verify_accept(tok, par, s["logits"], BLOCK, s["acc"], s["acc_nodes"], s["out"], s["aws"])
        bd.domino_target_commit(s["model"], tok.shape[1], s["lens"], s["acc"], s["acc_nodes"], s["ck"], s["cv"],
                                s["cap"], s["new_lens"], s["ws"])
        return dict(done, logits=s["logits"], new_lens=s["new_lens"], ck=s["ck"], cv=s["cv"])
    if kind == "accept":
        bd.domino_verify_accept(tok, par, s["logits"], BLOCK, s["acc"], s["acc_nodes"], s["out"], s["ws"])
    else:
        bd.domino_verify_sample(tok, s["logits"], s["draft"], case["temperature"], s["seed"], s["acc"], s["acc_nodes"],
                                s["out"], s["ws"])
    return done


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def _mean_ctx(case):
    return case["ctx"] * (0.625 if case["ragged"] and case["batch"] > 1 else 1.0)


def work(case):
    kind, b = case["kind"], case["batch"]
    if kind == "accept":
        nodes = BLOCK  # rows of the nodes with children, and the last one's
        return {"bytes": float(b * nodes * case["vocab"] * (2 if case["logits"] == "bf16" else 4)),
                "flops": float(b * nodes * case["vocab"])}
    if kind == "accept_sampled":
        per = 2 if case["logits"] == "bf16" else 4
        return {"bytes": float(b * case["vocab"] * (BLOCK * per + (BLOCK - 1) * 4)),
                "flops": float(4 * b * BLOCK * case["vocab"])}
    cfg = _cfg(case)
    e = 2 if cfg.dtype == "bf16" else 4
    qd, kvd, d = cfg.n_q_heads * cfg.head_dim, cfg.n_kv_heads * cfg.head_dim, cfg.hidden
    layer = d * (qd + 2 * kvd) + qd * d + 3 * d * cfg.ffn
    nodes = 1 + (BLOCK - 1) * case["branch"] if kind == "verify" else BLOCK
    lm_rows = nodes if kind == "verify" else BLOCK - 1
    ctx, n_new = _mean_ctx(case), case.get("n_new", 0)
    rows = b * nodes
    params = cfg.n_layers * layer + cfg.vocab * d
    flops = 2.0 * rows * cfg.n_layers * layer + 2.0 * b * lm_rows * cfg.vocab * d
    flops += 4.0 * rows * (ctx + nodes) * qd * cfg.n_layers
    byts = params * e + 2.0 * cfg.n_layers * b * ctx * kvd * e
    if kind != "verify":
        ds, r = cfg.gru_hidden, cfg.rank
        head = 3 * ds * (d + ds) + r * (d + ds) + cfg.vocab * r
        byts += head * e
        flops += 2.0 * b * (BLOCK - 1) * head
    else:
        byts += rows * cfg.vocab * (2.0 if case["logits"] == "bf16" else 4.0)
    if kind == "sampled":
        byts += 4.0 * b * (BLOCK - 1) * cfg.vocab
    if n_new:
        flops += 2.0 * b * n_new * (cfg.ctx_fuse_layers * d * d + 2 * cfg.n_layers * kvd * d)
        byts += cfg.ctx_fuse_layers * d * d * e + 4.0 * b * n_new * d * max(1, cfg.ctx_fuse_layers)
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    """About four times what the fp32 path shows against 64 bits: 1.6e-5 on a
    step's hidden rows, 5.6e-5 where keys and values were first rounded to a bf16
    cache, 4.1e-5 on the logits of 36 layers.  A value that is stored in bf16 may
    fall to the other side of a rounding (2^-8 of itself); whole values may
    differ at ties."""
    kind = case["kind"]
    if kind == "accept":
        return "exact"
    if kind == "accept_sampled":
        return {"rel": 0.0, "differ": 0.01}
    if kind == "verify":
        return {"rel": 1e-3 if case["logits"] == "bf16" else 2e-4, "max": 1e-2, "differ": 0.005}
    if case.get("n_new", 0):
        return {"rel": 2e-4, "max": 1e-2, "differ": 0.005}
    return {"rel": 7e-5, "max": 3e-3, "differ": 0.005}


# --------------------------------------------------------------------------
# the same outputs in 64 bits
# --------------------------------------------------------------------------
F64 = torch.float64


def _mm(x, w):
    """x @ w.T in 64 bits, the matrix widened a block of rows at a time."""
    return torch.cat([x @ part.to(F64).t() for part in w.split(16384)], dim=-1)


def _rms(x, g, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g.to(F64)


def _rope(x, pos, theta):
    half = x.shape[-1] // 2
    ang = pos.to(F64)[:, None, None] * torch.pow(torch.tensor(theta, dtype=F64, device=DEV),
                                                 -torch.arange(half, dtype=F64, device=DEV) / half)
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


def _layers(cfg, w, x, pos, lens, ck, cv, allow=None, keep=None):
    """x [b*n, d] through every layer; `allow` [b, n, n] limits the keys of the block itself."""
    b, nq, nkv, dh = lens.shape[0], cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim
    n, grp = x.shape[0] // b, nq // nkv
    for l, lw in enumerate(w["layers"]):
        a = _rms(x, lw["attn_norm"], cfg.rms_eps)
        q = _rope(_rms(_mm(a, lw["wq"]).view(-1, nq, dh), lw["q_norm"], cfg.rms_eps), pos, cfg.rope_theta)
        k = _rope(_rms(_mm(a, lw["wk"]).view(-1, nkv, dh), lw["k_norm"], cfg.rms_eps), pos, cfg.rope_theta)
        v = _mm(a, lw["wv"]).view(-1, nkv, dh)
        o = torch.empty((b * n, nq, dh), dtype=F64, device=DEV)
        for i in range(b):
            m, at = int(lens[i]), slice(i * n, (i + 1) * n)
            for h in range(nkv):
                keys = torch.cat([ck[l, i, :m, h].to(F64), k[at, h]])
                vals = torch.cat([cv[l, i, :m, h].to(F64), v[at, h]])
                qs = q[at, h * grp:(h + 1) * grp].transpose(0, 1).reshape(grp * n, dh)
                sc = qs @ keys.t() / math.sqrt(dh)
                if allow is not None:
                    sc[:, m:].masked_fill_(~allow[i].repeat(grp, 1), -math.inf)
                o[at, h * grp:(h + 1) * grp] = (sc.softmax(-1) @ vals).view(grp, n, dh).transpose(0, 1)
        if keep is not None:
            keep.append((k, v))
        x = x + _mm(o.view(b * n, nq * dh), lw["wo"])
        y = _rms(x, lw["ffn_norm"], cfg.rms_eps)
        x = x + _mm(torch.nn.functional.silu(_mm(y, lw["w_gate"])) * _mm(y, lw["w_up"]), lw["w_down"])
    return _rms(x, w["final_norm"], cfg.rms_eps)


def _words(seed, row, depth, n):
    """The first n words of the draft noise of (row, depth): Philox-4x32-10."""
    low = 0xFFFFFFFF
    c = [torch.arange(-(-n // 4), dtype=torch.int64, device=DEV)]
    c += [torch.full_like(c[0], x) for x in (depth, row, 0)]
    k0, k1 = seed & low, (seed >> 32) & low
    for r in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [(p1 >> 32) & low ^ c[1] ^ k0, p1 & low, (p0 >> 32) & low ^ c[3] ^ k1, p0 & low]
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    return torch.stack(c, -1).reshape(-1)[:n]


def _exact_drafter(case, cfg, seed, s):
    kind, b, w = case["kind"], case["batch"], _weights(cfg, seed)
    lens, n = s["lens"], case.get("n_new", 0)
    ck, cv = s["ck"], s["cv"]
    if n:
        ck, cv = ck.to(F64), cv.to(F64)
        c = s["new"].view(b * n, -1).to(F64)
        c = _mm(c, w["ctx_fc"]) if cfg.ctx_fuse_layers else c
        at = (lens[:, None] - n + torch.arange(n, device=DEV)).long()
        rows = torch.arange(b, device=DEV)[:, None].expand(b, n)
        for l, lw in enumerate(w["layers"]):
            k = _rms(_mm(c, lw["wk"]).view(b * n, -1, cfg.head_dim), lw["k_norm"], cfg.rms_eps)
            ck[l, rows, at] = _rope(k, at.reshape(-1), cfg.rope_theta).view(b, n, -1, cfg.head_dim)
            cv[l, rows, at] = _mm(c, lw["wv"]).view(b, n, -1, cfg.head_dim)
        if cfg.dtype == "bf16":  # a cache holds its storage type
            ck, cv = ck.to(torch.bfloat16), cv.to(torch.bfloat16)
    tok = torch.full((b, BLOCK), cfg.mask_id, dtype=torch.int64, device=DEV)
    tok[:, 0] = s["anchor"]
    pos = (lens[:, None] + torch.arange(BLOCK, device=DEV)).view(-1)
    x = _layers(cfg, w, w["embed"][tok.view(-1)].to(F64), pos, lens, ck, cv)
    h = x.view(b, BLOCK, -1)[:, 1:].contiguous()
    base = _mm(h.view(-1, cfg.hidden), w["lm_head"]).view(b, BLOCK - 1, -1)
    state, y = torch.zeros((b, cfg.gru_hidden), dtype=F64, device=DEV), s["anchor"].long()
    w2, beta = w["w2"].to(F64), case.get("branch", 1)
    ids, vals, ces, finals = [], [], [], []
    for j in range(BLOCK - 1):
        gi = _mm(w["embed"][y].to(F64), w["gru_w_ih"]) + w["gru_b_ih"].to(F64)
        gh = _mm(state, w["gru_w_hh"]) + w["gru_b_hh"].to(F64)
        (ir, iz, ic), (hr, hz, hc) = gi.chunk(3, -1), gh.chunk(3, -1)
        z = torch.sigmoid(iz + hz)
        state = (1 - z) * torch.tanh(ic + torch.sigmoid(ir + hr) * hc) + z * state
        u = torch.nn.functional.silu(_mm(torch.cat([h[:, j], state], -1), w["w1"]))
        final = base[:, j] + u @ w2.t()
        if kind == "train":
            y = s["labels"][:, j].long()
            ces.append(torch.stack([torch.logsumexp(t, -1) - t.gather(1, y[:, None])[:, 0] for t in (base[:, j], final)]))
            continue
        if kind == "sampled":
            finals.append(final)
            noise = torch.stack([_words(case_seed(seed), i, j + 1, cfg.vocab) for i in range(b)])
            uni = ((noise >> 9).to(F64) + 0.5) / 2.0 ** 23
            ids.append((final / case["temperature"] - uni.log().neg().log()).argmax(-1, keepdim=True))
        else:
            ids.append(final.topk(beta, -1).indices)
        vals.append(final.gather(1, ids[-1]))
        y = ids[-1][:, 0]
    if kind == "train":
        ce = torch.stack(ces, -1)
        wk = torch.exp(-torch.arange(BLOCK - 1, dtype=F64, device=DEV) / 15.0)
        base_l, final_l = ((ce * wk).sum((1, 2)) / (b * wk.sum())).tolist()
        loss = torch.tensor([0.5 * final_l + 0.5 * base_l, base_l, final_l], dtype=F64)
        return dict(loss=loss, ce=ce, hidden=h)
    out = dict(ids=None, vals=torch.stack(vals, 1), hidden=h, tokens=None, parents=None, depths=None, positions=None,
               mask=None)
    if kind == "sampled":
        out["final_logits"] = torch.stack(finals, 1)
    if n:
        out.update(ck=ck, cv=cv)
    return out


def case_seed(seed):
    """The seed of the draws of a sampled case."""
    return seed + 77


def exact(case, seed):
    kind = case["kind"]
    if kind in ("accept", "accept_sampled"):
        return None  # whole numbers only
    cfg = _cfg(case)
    s = _context(case, cfg, seed)
    if kind != "verify":
        if kind == "train":
            s["labels"] = torch.randint(0, cfg.vocab, (case["batch"], BLOCK - 1), generator=_gen(seed, 5), device=DEV,
                                        dtype=torch.int32)
        return _exact_drafter(case, cfg, seed, s)
    w = _weights(cfg, seed, head=False)
    tok, _, _, pos, mask = _random_tree(case, seed, cfg.vocab, s["anchor"], s["lens"])
    b, nn = tok.shape
    keep = []
    x = _layers(cfg, w, w["embed"][tok.view(-1).long()].to(F64), pos.view(-1), s["lens"], s["ck"], s["cv"],
                allow=mask.bool(), keep=keep)
    logits = _mm(x, w["lm_head"]).view(b, nn, -1)
    return dict(accept_len=None, accepted_nodes=None, out_tokens=None, logits=logits, new_lens=None, ck=None, cv=None)
