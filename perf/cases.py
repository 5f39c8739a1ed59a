"""The calls a drafting program makes of this library, at the sizes it makes them: what the performance of the
repository is measured on.

A case is one of
  draft    one fuzzy forward (easyspec_draft_step) of every live sequence; the common call of the whole method
  tree     two levels of a token tree (easyspec_draft_tree_step), the second hanging below the first
  calib    one bonus calibration or one chunk of a prompt prefill (easyspec_calibrate), `tokens` per sequence
  loop     one drafting iteration without its acceptance: a calibration, then `steps` fuzzy steps
  accept   acceptance by speculative sampling of `batch` sequences (easyspec_accept)
  kv       a sequence's cache taken in and handed out again (easyspec_kv_import, easyspec_kv_export): prefix reuse
The models are the repository's own shapes with random parameters drawn on the device by the repository's recipe
(projections, embedding and biases N(0, 0.02^2), gains 1 + N(0, 0.02^2), a KV prefix of N(0, 1)), whole or at reduced
depth and vocabulary.  Token ids are uniform and given, not fed back, so that a tie cannot change the work.
"""
import math

import numpy as np
import torch

import easyspec_synth as synth
import paper_2502_02493_amd as es

DEV = "cuda:0"
TREE_W = es.EASYSPEC_MAX_TREE_WIDTH


# ----------------------------------------------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------------------------------------------

def _model(kind, model, contexts, dtype=None, layers=0, vocab=0, group=4, policy="aligned", full_layer=False, tokens=1,
           all_rows=False, steps=1, width=4, width2=8):
    shape = synth.model_shape(model)
    c = dict(kind=kind, model=model, dtype=dtype or shape["dtype"], layers=layers or shape["n_layers"],
             vocab=vocab or shape["vocab"], contexts=",".join(str(n) for n in contexts))
    if kind in ("draft", "tree", "loop"):
        c.update(group=group, policy=policy, full_layer=full_layer)
    if kind in ("calib", "loop"):
        c.update(tokens=",".join(str(n) for n in (tokens if isinstance(tokens, list) else [tokens] * len(contexts))))
    if kind == "calib":
        c.update(all_rows=all_rows)
    if kind == "loop":
        c.update(steps=steps)
    if kind == "tree":
        c.update(width=width, width2=width2)
    return c


def listed():
    return [
        # the smallest drafter in use (fp32, four layers): launches and latency, hardly any bytes
        dict(_model("draft", "tiny", [128], group=2, policy="packed"), name="draft_tiny_fp32"),
        # a whole small iteration of odd shapes: 448 wide, 7 heads per KV head, 1184 hidden, 1000 words, with biases
        dict(_model("loop", "tiny_qwen", [61], group=2, policy="packed", tokens=5, steps=3), name="loop_tiny_qwen_fp32"),
        # the headline call: one fuzzy step of the 8B drafter after a 2048-token context
        dict(_model("draft", "llama3_8b", [2048]), name="draft_8b"),
        # the calibration that follows five accepted drafts
        dict(_model("calib", "llama3_8b", [2048], tokens=6), name="calib_8b_6"),
        # one full chunk of a long prompt
        dict(_model("calib", "llama3_8b", [8192], tokens=16), name="prefill_8b_16"),
        # the second shape: 7 query heads per KV head, biases, d_ffn that is no multiple of the batch of the weight stream
        dict(_model("draft", "qwen2_7b", [4096]), name="draft_qwen7b"),
        # a token tree growing by a narrow and a wide level
        dict(_model("tree", "llama3_8b", [2048], width=4, width2=12), name="tree_8b_4_12"),
        # four users at long contexts share one step ...
        dict(_model("draft", "llama3_8b", [4096, 8192, 16384, 32768]), name="draft_8b_batch4_long"),
        # ... and the calibration after it
        dict(_model("calib", "llama3_8b", [4096, 8192, 16384, 32768], tokens=6), name="calib_8b_batch4"),
        # sixteen users prefill a full chunk each: the most tokens one call takes
        dict(_model("calib", "llama3_8b", [512 + 37 * i for i in range(16)], tokens=16), name="prefill_8b_16x16"),
        # sampling acceptance of one sequence at the paper's speculation length and second temperature
        dict(kind="accept", batch=1, gamma=5, vocab=128256, temperature=0.8, name="accept_8b"),
        # a prompt prefix of 2048 slots taken from a store into the cache and back out
        dict(_model("kv", "llama3_8b", [2048]), name="kv_8b"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["draft", "draft", "tree", "calib", "calib", "calib", "loop", "accept", "kv"])
    if kind == "accept":
        return dict(kind="accept", batch=_log_int(rng, 1, 16), gamma=rng.randint(1, 10), vocab=_log_int(rng, 900, 152064),
                    temperature=round(rng.uniform(0.5, 1.2), 2))
    model = rng.choice(["tiny", "tiny_qwen", "llama3_8b", "llama3_8b", "qwen2_7b", "qwen2_7b"])
    small = model.startswith("tiny")
    dtype = rng.choice(["fp32", "bf16"]) if small else rng.choice(["bf16", "bf16", "bf16", "fp32"])
    layers = rng.randint(2, 8) if small else rng.randint(2, 4) if dtype == "fp32" else _log_int(rng, 2, 8 if kind == "loop" else 20)
    vocab = _log_int(rng, 500, 8000) if small else _log_int(rng, 1000, 152064)
    batch = 1 if kind == "tree" or rng.random() < 0.4 else _log_int(rng, 2, 16)
    most = 600 if small else min(16384, 40000 // batch)
    contexts = [_log_int(rng, 16, most) for _ in range(batch)]
    if kind == "kv":
        contexts = contexts[:1]
    t = rng.randint(1, 16)  # tokens of a calibration: the same for all sequences, or up to that many each
    tokens = [rng.randint(1, t) for _ in contexts] if rng.random() < 0.5 else t
    return _model(kind, model, contexts, dtype=dtype, layers=layers, vocab=vocab, group=rng.randint(1, 8),
                  policy=rng.choice(["aligned", "packed"]), full_layer=rng.random() < 0.15, tokens=tokens,
                  all_rows=rng.random() < 0.3, steps=rng.randint(1, 4), width=rng.randint(1, 6), width2=rng.randint(1, 16))


# ----------------------------------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------------------------------

def _shape(case):
    return synth.model_shape(case["model"], n_layers=case["layers"], vocab=case["vocab"], dtype=case["dtype"])


def _contexts(case):
    return [int(n) for n in case["contexts"].split(",")]


def _n_tokens(case):
    return [int(n) for n in case["tokens"].split(",")]


def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(1000003 * int(seed) + salt)


def _weights(case, seed):
    """Parameters on the device, in the layout of easyspec_load_weights."""
    cfg, gen = _shape(case), _gen(seed, 1)
    dt = torch.bfloat16 if cfg["dtype"] == "bf16" else torch.float32
    d, f, v, hd = cfg["d_model"], cfg["d_ffn"], cfg["vocab"], cfg["head_dim"]
    hq, hkv = cfg["n_q_heads"] * hd, cfg["n_kv_heads"] * hd

    def mat(rows, cols):
        return torch.empty(rows, cols, dtype=dt, device=DEV).normal_(0.0, 0.02, generator=gen)

    def vec(n, mean):
        return torch.empty(n, dtype=torch.float32, device=DEV).normal_(mean, 0.02, generator=gen).to(dt).float()

    layers = []
    for _ in range(cfg["n_layers"]):
        w = dict(wq=mat(hq, d), wk=mat(hkv, d), wv=mat(hkv, d), wo=mat(d, hq), wg=mat(f, d), wu=mat(f, d), wd=mat(d, f),
                 g_attn=vec(d, 1.0), g_mlp=vec(d, 1.0))
        if cfg["qkv_bias"]:
            w.update(bq=vec(hq, 0.0), bk=vec(hkv, 0.0), bv=vec(hkv, 0.0))
        layers.append(w)
    return dict(layers=layers, embed=mat(v, d), lm_head=mat(v, d), g_final=vec(d, 1.0))


def _prefix(case, seed, b):
    """The prefilled context of sequence b: K and V, [layer][KV head][slot][head_dim] in the storage type."""
    cfg, gen = _shape(case), _gen(seed, 100 + b)
    dt = torch.bfloat16 if cfg["dtype"] == "bf16" else torch.float32
    shape = (cfg["n_layers"], cfg["n_kv_heads"], _contexts(case)[b], cfg["head_dim"])
    return [torch.empty(shape, dtype=dt, device=DEV).normal_(0.0, 1.0, generator=gen) for _ in range(2)]


def _tokens(case, seed, shape):
    return torch.randint(0, case["vocab"], shape, dtype=torch.int32, device=DEV, generator=_gen(seed, 7))


def _parents(case):
    """Two tree levels: the first hangs off the context, the second's nodes are spread over the first's."""
    w, w2 = case["width"], case["width2"]
    return [-1] * w, [i * w // w2 for i in range(w2)]


def _tree_row(par):
    row = np.full((1, TREE_W), -1, np.int32)
    row[0, : len(par)] = par
    return row


class _Ctx:
    """The handle a program keeps; given back with the state."""

    def __init__(self, case):
        self.lens = _contexts(case)
        n_max = max(self.lens) + 64
        self.h = es.easyspec_create(es.make_config(_shape(case), len(self.lens), n_max, 16), torch.cuda.current_stream().cuda_stream)

    def rewind(self):
        """Back to the prefix: what a program does when it drops what it drafted (host state only)."""
        for b, n in enumerate(self.lens):
            es.easyspec_truncate(self.h, b, n)

    def __del__(self):
        if getattr(self, "h", None) is not None:
            es.easyspec_destroy(self.h)
            self.h = None


def _accept_inputs(case, seed):
    B, g, V, T = case["batch"], case["gamma"], case["vocab"], case["temperature"]
    gen = _gen(seed, 3)
    target = torch.empty(B, g + 1, V, device=DEV).normal_(0.0, 2.0, generator=gen)
    draft_logits = target[:, :g] + 0.5 * torch.empty(B, g, V, device=DEV).normal_(0.0, 1.0, generator=gen)
    # drafted tokens drawn from the draft's own distribution (Gumbel maximum)
    noise = torch.rand(B, g, V, device=DEV, generator=gen).clamp_(1e-20, 1.0)
    draft = (draft_logits / T - torch.log(-torch.log(noise).clamp_min_(1e-20))).argmax(-1).to(torch.int32).contiguous()
    return dict(draft=draft, draft_logits=draft_logits.contiguous(), target_logits=target.contiguous(),
                r=torch.rand(B, g, device=DEV, generator=gen), u=torch.rand(B, device=DEV, generator=gen))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "accept":
        st = _accept_inputs(case, seed)
        ws = es.easyspec_accept_workspace_bytes(case["batch"], case["gamma"], case["vocab"])
        st.update(case=case, ws=torch.empty((ws + 7) // 8, dtype=torch.float64, device=DEV),
                  acc=torch.zeros(case["batch"], dtype=torch.int32, device=DEV),
                  bonus=torch.zeros(case["batch"], dtype=torch.int32, device=DEV))
        return st
    ctx = _Ctx(case)
    B, V, lens = len(ctx.lens), case["vocab"], ctx.lens
    st = dict(case=case, ctx=ctx)
    if kind == "kv":
        k, v = _prefix(case, seed, 0)
        st.update(k=k, v=v, k_out=torch.zeros_like(k), v_out=torch.zeros_like(v))
        return st
    es.easyspec_load_weights(ctx.h, _weights(case, seed))
    for b in range(B):
        k, v = _prefix(case, seed, b)
        es.easyspec_kv_import(ctx.h, b, k, v, lens[b])
    if kind in ("draft", "tree", "loop"):
        policy = es.EASYSPEC_POLICY_ALIGNED if case["policy"] == "aligned" else es.EASYSPEC_POLICY_PACKED
        es.easyspec_set_groups(ctx.h, es.easyspec_default_groups(case["layers"], case["group"], policy))
        if case["full_layer"]:
            es.easyspec_set_parallel_mode(ctx.h, es.EASYSPEC_PARALLEL_FULL_LAYER)

    def out(*shape):
        return torch.zeros(*shape, V, dtype=torch.float32, device=DEV), torch.zeros(*shape, dtype=torch.int32, device=DEV)

    if kind == "draft":
        st["tok"] = _tokens(case, seed, (B,))
        st["logits"], st["next"] = out(B)
    elif kind == "tree":
        st["tok"] = _tokens(case, seed, (2, 1, TREE_W))
        st["logits"], st["next"] = zip(out(1, TREE_W), out(1, TREE_W))
        st["n"] = [np.array([case["width"]], np.int32), np.array([case["width2"]], np.int32)]
        st["parents"] = [_tree_row(p) for p in _parents(case)]
    else:
        st["tok"] = _tokens(case, seed, (B, 16))
        st["n"] = np.array(_n_tokens(case), np.int32)
        rows = kind == "calib" and case["all_rows"]
        st["logits"] = [torch.zeros(B, 16, V, device=DEV) if rows else torch.zeros(B, V, device=DEV)]
        st["next"] = [torch.zeros(B, dtype=torch.int32, device=DEV)]
        if kind == "loop":
            st["step_tok"] = torch.randint(0, V, (case["steps"], B), dtype=torch.int32, device=DEV, generator=_gen(seed, 8))
            for _ in range(case["steps"]):
                lg, nx = out(B)
                st["logits"].append(lg)
                st["next"].append(nx)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "accept":
        es.easyspec_accept(st["draft"], st["draft_logits"], st["target_logits"], st["r"], st["u"], case["batch"], case["gamma"],
                           case["vocab"], case["temperature"], st["acc"], st["bonus"], st["ws"], torch.cuda.current_stream().cuda_stream)
        return [st["acc"], st["bonus"]]
    ctx = st["ctx"]
    if kind == "kv":
        n = ctx.lens[0]
        es.easyspec_kv_import(ctx.h, 0, st["k"], st["v"], n)
        es.easyspec_kv_export(ctx.h, 0, st["k_out"], st["v_out"], n)
        return [st["k_out"], st["v_out"]]
    ctx.rewind()
    if kind == "draft":
        es.easyspec_draft_step(ctx.h, st["tok"], st["next"], st["logits"])
        return [st["logits"], st["next"]]
    if kind == "tree":
        for i in range(2):
            es.easyspec_draft_tree_step(ctx.h, st["tok"][i], st["n"][i], st["parents"][i], st["next"][i], st["logits"][i])
        return list(st["logits"]) + list(st["next"])
    rows = 1 if kind == "calib" and case["all_rows"] else 0
    es.easyspec_calibrate(ctx.h, st["tok"], st["n"], st["next"][0], st["logits"][0], rows)
    if kind == "loop":
        for i in range(case["steps"]):
            es.easyspec_draft_step(ctx.h, st["step_tok"][i], st["next"][i + 1], st["logits"][i + 1])
    return st["logits"] + st["next"]


# ----------------------------------------------------------------------------------------------------------------
# the work, the tolerance
# ----------------------------------------------------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "accept":
        B, g, V = case["batch"], case["gamma"], case["vocab"]
        return {"bytes": 4.0 * B * ((2 * g + 1) * V + 3 * g + 3), "flops": 2.0 * B * (2 * g + 1) * V}
    cfg, lens = _shape(case), _contexts(case)
    e = 2 if cfg["dtype"] == "bf16" else 4
    L, d, f, V, hd = cfg["n_layers"], cfg["d_model"], cfg["d_ffn"], cfg["vocab"], cfg["head_dim"]
    hq, hkv = cfg["n_q_heads"] * hd, cfg["n_kv_heads"] * hd
    slot = 2 * L * hkv * e  # K and V of one slot in every layer
    if kind == "kv":
        return {"bytes": 4.0 * slot * lens[0], "flops": 0.0}  # taken in, written, read, handed out
    per_layer = (hq + 2 * hkv) * d + d * hq + 3 * f * d
    B = len(lens)

    def forward(cols, rows_out, logit_rows):
        """One forward: cols = (slots read, columns of the sequence) per sequence."""
        n = sum(m for _, m in cols)
        attn = sum(4.0 * hq * L * s * m for s, m in cols)
        b = (per_layer * L + V * d) * e + sum(slot * s for s, _ in cols) + slot * n + n * d * e + 4.0 * logit_rows * V
        return b, 2.0 * (per_layer * L * n + V * d * rows_out) + attn

    if kind == "draft":
        parts = [forward([(n, 1) for n in lens], B, B)]
    elif kind == "tree":
        w, w2 = case["width"], case["width2"]
        parts = [forward([(lens[0], w)], w, w), forward([(lens[0] + w, w2)], w2, w2)]
    else:
        t = _n_tokens(case)
        rows = sum(t) if kind == "calib" and case["all_rows"] else B
        parts = [forward(list(zip(lens, t)), rows, rows)]
        if kind == "loop":
            parts += [forward([(n + m + i, 1) for n, m in zip(lens, t)], B, B) for i in range(case["steps"])]
    return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}


def tolerance(case):
    if case["kind"] in ("accept", "kv"):
        return "exact"
    # bf16: weights and cache in bf16, activations in two bf16 terms; what differs between two correct orders of
    # summation is now and then the last bit of a cache entry, which travels through the layers that follow
    # (measured against exact(): 1e-5 to 2.2e-4, fp32 5e-7 to 2.6e-6; about four times the largest)
    rel = 8e-4 if case["dtype"] == "bf16" else 1e-5
    return {"rel": rel, "max": 6 * rel, "differ": 0.05}


# ----------------------------------------------------------------------------------------------------------------
# the same in 64 bits, by plain torch
# ----------------------------------------------------------------------------------------------------------------

def _norm(x, gain, eps):
    return x * torch.rsqrt(x.pow(2).mean(-1, keepdim=True) + eps) * gain.double()


class _Exact:
    def __init__(self, case, seed):
        self.cfg = _shape(case)
        self.w = _weights(case, seed)
        self.lens = _contexts(case)
        self.kv = [_prefix(case, seed, b) for b in range(len(self.lens))]
        self.new = {}  # (sequence, layer) -> K, V of the slots after the prefix, [KV head][slot][head_dim]
        hd = self.cfg["head_dim"]
        self.freq = self.cfg["rope_theta"] ** (-2.0 * torch.arange(hd // 2, device=DEV, dtype=torch.float64) / hd)

    def rope(self, x, pos):  # [n][heads][hd]
        ang = pos.double()[:, None, None] * self.freq
        c, s = torch.cos(ang), torch.sin(ang)
        lo, hi = x.chunk(2, -1)
        return torch.cat([lo * c - hi * s, hi * c + lo * s], -1)

    def store(self, x):
        return x.to(torch.bfloat16).double() if self.cfg["dtype"] == "bf16" else x.float().double()

    def attn(self, l, h, cols):
        """cols: per sequence (b, tokens, rotary positions, visible[n][slots after the prefix incl. the new ones], kept)."""
        cfg, w = self.cfg, self.w["layers"][l]
        hq, hkv, hd = cfg["n_q_heads"], cfg["n_kv_heads"], cfg["head_dim"]
        x = _norm(h, w["g_attn"], cfg["rms_eps"])
        q, k, v = x @ w["wq"].double().t(), x @ w["wk"].double().t(), x @ w["wv"].double().t()
        if cfg["qkv_bias"]:
            q, k, v = q + w["bq"].double(), k + w["bk"].double(), v + w["bv"].double()
        outs, at = [], 0
        for b, tok, pos, vis, kept in cols:
            n = len(tok)
            qs = self.rope(q[at:at + n].view(n, hq, hd), pos)
            ks = self.store(self.rope(k[at:at + n].view(n, hkv, hd), pos)).transpose(0, 1)
            vs = self.store(v[at:at + n].view(n, hkv, hd)).transpose(0, 1)
            at += n
            if kept and (b, l) in self.new:
                ks, vs = torch.cat([self.new[b, l][0][:, :kept], ks], 1), torch.cat([self.new[b, l][1][:, :kept], vs], 1)
            self.new[b, l] = (ks, vs)
            K = torch.cat([self.kv[b][0][l].double(), ks], 1).contiguous()
            Vv = torch.cat([self.kv[b][1][l].double(), vs], 1).contiguous()
            g = hq // hkv
            qg = qs.view(n, hkv, g, hd).permute(1, 2, 0, 3).reshape(hkv, g * n, hd).contiguous()
            s = torch.matmul(qg, K.transpose(1, 2).contiguous()) / math.sqrt(hd)
            mask = torch.cat([torch.ones(n, self.lens[b], dtype=torch.bool, device=DEV), vis], 1)
            s = s.masked_fill(~mask.repeat(g, 1)[None], -math.inf)
            o = torch.matmul(torch.softmax(s, -1), Vv)
            outs.append(o.view(hkv, g, n, hd).permute(2, 0, 1, 3).reshape(n, hq * hd))
        return torch.cat(outs) @ w["wo"].double().t()

    def mlp(self, l, h):
        w = self.w["layers"][l]
        x = _norm(h, w["g_mlp"], self.cfg["rms_eps"])
        return (torch.nn.functional.silu(x @ w["wg"].double().t()) * (x @ w["wu"].double().t())) @ w["wd"].double().t()

    def forward(self, cols, bounds, full_layer=False):
        tok = torch.cat([c[1] for c in cols]).long()
        h = self.w["embed"][tok].double()
        for lo, hi in zip(bounds[:-1], bounds[1:]):
            a = [self.attn(l, h, cols) for l in range(lo, hi)]
            if full_layer:
                h = h + sum(a) + sum(self.mlp(l, h + a[l - lo]) for l in range(lo, hi))
            else:
                for l in range(lo, hi):
                    h = h + a[l - lo]
                    h = h + self.mlp(l, h)
        x = _norm(h, self.w["g_final"], self.cfg["rms_eps"])
        return torch.cat([x @ p.double().t() for p in self.w["lm_head"].split(16384)], -1)


def _exact_accept(case, seed):
    x = _accept_inputs(case, seed)
    T, g = case["temperature"], case["gamma"]
    acc, bonus = [], []
    for b in range(case["batch"]):
        p = torch.softmax(x["target_logits"][b].double() / T, -1)
        pd = torch.softmax(x["draft_logits"][b].double() / T, -1)
        m = 0
        while m < g and not float(x["r"][b, m].double() * pd[m, x["draft"][b, m].long()]) > float(p[m, x["draft"][b, m].long()]):
            m += 1
        q = (p[m] - pd[m]).clamp_min(0.0) if m < g else p[g]
        run_sum = torch.cumsum(q, 0)
        acc.append(m)
        bonus.append(int((run_sum > x["u"][b].double() * run_sum[-1]).int().argmax()))
    return [torch.tensor(acc, dtype=torch.int32), torch.tensor(bonus, dtype=torch.int32)]


def exact(case, seed):
    kind = case["kind"]
    if kind == "accept":
        return _exact_accept(case, seed)
    if kind == "kv":
        return [x.double() for x in _prefix(case, seed, 0)]  # nothing is computed: what went in comes out
    m = _Exact(case, seed)
    L, V, lens = case["layers"], case["vocab"], m.lens
    B = len(lens)
    single = list(range(L + 1))
    bounds = single
    if kind != "calib":
        policy = es.EASYSPEC_POLICY_ALIGNED if case["policy"] == "aligned" else es.EASYSPEC_POLICY_PACKED
        bounds = [int(x) for x in es.easyspec_default_groups(L, case["group"], policy)]
    full = kind != "calib" and case["full_layer"]

    def causal(n, before):
        return torch.ones(n, before + n, dtype=torch.bool, device=DEV).tril(before)

    def at(b, first, n):
        return torch.arange(lens[b] + first, lens[b] + first + n, device=DEV)

    if kind == "draft":
        tok = _tokens(case, seed, (B,))
        return [m.forward([(b, tok[b:b + 1], at(b, 0, 1), causal(1, 0), 0) for b in range(B)], bounds, full), None]
    if kind == "tree":
        tok = _tokens(case, seed, (2, 1, TREE_W))
        w, w2 = case["width"], case["width2"]
        par = _parents(case)[1]
        outs = []
        for i, n in enumerate((w, w2)):
            vis = torch.zeros(n, w * i + n, dtype=torch.bool, device=DEV)
            for j in range(n):
                vis[j, w * i + j] = True
                if i:
                    vis[j, par[j]] = True
            pos = torch.full((n,), lens[0] + i, device=DEV)
            lg = m.forward([(0, tok[i, 0, :n], pos, vis, w * i)], bounds, full)
            whole = torch.zeros(1, TREE_W, V, dtype=torch.float64, device=DEV)
            whole[0, :n] = lg
            outs.append(whole)
        return outs + [None, None]
    t = _n_tokens(case)
    tok = _tokens(case, seed, (B, 16))
    rows = m.forward([(b, tok[b, :n], at(b, 0, n), causal(n, 0), 0) for b, n in enumerate(t)], single).split(t)
    if kind == "calib" and case["all_rows"]:
        whole = torch.zeros(B, 16, V, dtype=torch.float64, device=DEV)
        for b, n in enumerate(t):
            whole[b, :n] = rows[b]
        return [whole, None]
    outs = [torch.stack([r[-1] for r in rows])]
    if kind == "loop":
        step_tok = torch.randint(0, V, (case["steps"], B), dtype=torch.int32, device=DEV, generator=_gen(seed, 8))
        for i in range(case["steps"]):
            outs.append(m.forward([(b, step_tok[i, b:b + 1], at(b, n + i, 1), causal(1, n + i), n + i) for b, n in enumerate(t)],
                                  bounds, full))
    return outs + [None] * len(outs)
