"""The work whose time counts in this framework, as cases: one pass each through the public entry points
of paper_2404_18911_amd.binding, at the shapes of inputs.SHAPES (whole models, or fewer layers of the same
width where one layer more only repeats the work).

Kinds of cases:
  linear    kg_op_linear: one weight-streaming projection of 1..8 rows, the unit every decode forward is made of
  prefill   kg_prefill: the prompt pass; returns the next token, its logits and the whole key / value cache
  plain     kg_prefill of a prompt, then kg_plain_step along a given continuation, logits of every step
            (scoring a continuation, or a caller that draws its own tokens)
  kangaroo  kg_generate: a whole request through the draft-and-verify loop, greedy or sampling
  train     kg_train_step on tokens: frozen model, adapter forward and backward, AdamW; returns the gradients
  features  kg_train_accumulate_features + kg_train_apply: the same step from a sequence's stored features

Weights are random, drawn on the GPU from the seed, and have one property of a trained model that a plain
random one lacks: a next token that stands out.  The row of the LM head for token next(v) is a multiple of
the embedding of v, so a position whose token is v prefers next(v) by far more than rounding can move, and the
tokens of a run do not depend on the order of a sum.  For a share of the tokens (`weak`) that row is scaled
down until the token still comes first but with little probability, so drafting stops there (confidence
below eta) and draft lengths vary as they do in real use.  Layers from the exit layer on and the adapter have
their output projections scaled by alpha = 0.1 as in inputs.py.
"""
import math

import numpy as np
import torch

from paper_2404_18911_amd import binding as B
from paper_2404_18911_amd import inputs as I

ALPHA, STD, ETA, GAMMA = 0.1, 0.02, 0.6, 6
PAGE = 128


def listed():
    return [
        # the smallest call: one row through one square projection (o_proj of the 7B shape): latency and launches
        {"name": "linear_1x4096x4096", "kind": "linear", "M": 1, "N": 4096, "K": 4096, "dtype": "bf16"},
        # seven verification rows through a wide projection of uneven sizes (no power of two, k not a multiple of 32)
        {"name": "linear_7x13840x5136", "kind": "linear", "M": 7, "N": 13840, "K": 5136, "dtype": "bf16"},
        # a whole request on the small float32 model: 16 prompt tokens, 32 new ones; bound by launches and the host
        {"name": "kangaroo_toy_f32", "kind": "kangaroo", "shape": "toy", "layers": 4, "tokens": 16, "new": 32, "weak": 0.4,
         "mode": 0, "adapter": 0, "kv": ""},
        # a short question to the 7B model: the whole prompt pass
        {"name": "prefill_7b_45", "kind": "prefill", "shape": "7b", "layers": 32, "tokens": 45, "adapter": 0, "kv": ""},
        # the prompt of the benchmark
        {"name": "prefill_7b_256", "kind": "prefill", "shape": "7b", "layers": 32, "tokens": 256, "adapter": 0, "kv": ""},
        # the long-context prompt, the largest case
        {"name": "prefill_7b_4096", "kind": "prefill", "shape": "7b", "layers": 32, "tokens": 4096, "adapter": 0, "kv": ""},
        # an uneven prompt at the 13B width
        {"name": "prefill_13b_777", "kind": "prefill", "shape": "13b", "layers": 6, "tokens": 777, "adapter": 0, "kv": ""},
        # one token at a time through the whole 7B model
        {"name": "plain_7b", "kind": "plain", "shape": "7b", "layers": 32, "tokens": 31, "new": 32, "adapter": 0, "kv": ""},
        # the headline: a greedy Kangaroo request on the 7B shape
        {"name": "kangaroo_7b", "kind": "kangaroo", "shape": "7b", "layers": 32, "tokens": 64, "new": 96, "weak": 0.5,
         "mode": 0, "adapter": 0, "kv": ""},
        # long context, speculative sampling at temperature 1: attention over thousands of cached positions
        {"name": "kangaroo_7b_ctx4000_sampling", "kind": "kangaroo", "shape": "7b", "layers": 6, "tokens": 4000, "new": 150,
         "weak": 0.0, "mode": 1, "adapter": 0, "kv": ""},
        # one training step of the adapter on a 256-token sequence
        {"name": "train_7b_256", "kind": "train", "shape": "7b", "layers": 32, "tokens": 256, "adapter": 0, "kv": ""},
        # an epoch over stored features: a longer, uneven sequence
        {"name": "features_7b_1000", "kind": "features", "shape": "7b", "layers": 2, "tokens": 1000, "adapter": 0, "kv": ""},
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "prefill", "prefill", "prefill", "plain", "kangaroo", "kangaroo", "train", "features"])
    if kind == "linear":
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        top = 2048 if dtype == "bf16" else 128
        return {"kind": kind, "M": rng.randint(1, 8), "N": 16 * _log(rng, 16, top), "K": 16 * _log(rng, 16, 1024 if dtype == "bf16" else 64),
                "dtype": dtype}
    shape = rng.choice(["7b", "7b", "13b", "33b"])
    adapter = rng.choice([0, 0, 0, 1, 2, 3])
    kv = rng.choice(["", "", "", "", "bf16", "f32"])
    layers = rng.randint(4, 6)
    if kind == "prefill":
        return {"kind": kind, "shape": shape, "layers": layers, "tokens": _log(rng, 2, 5000 if kv == "" else 1500), "adapter": adapter, "kv": kv}
    if kind == "plain":
        return {"kind": kind, "shape": shape, "layers": layers, "tokens": _log(rng, 2, 1500), "new": rng.randint(8, 40), "adapter": 0, "kv": kv}
    if kind == "kangaroo":
        shape = rng.choice(["toy", "small_bf16", "7b", "13b"])
        if shape in ("toy", "small_bf16"):
            layers, kv = I.SHAPES[shape].n_layers, ""
        return {"kind": kind, "shape": shape, "layers": layers, "tokens": _log(rng, 4, 300 if shape == "toy" else 3000), "new": rng.randint(20, 100),
                "weak": 0.0 if rng.random() < 0.3 else round(rng.uniform(0.2, 0.7), 2), "mode": 0, "adapter": adapter, "kv": kv}
    if kind == "train":
        return {"kind": kind, "shape": "7b", "layers": layers, "tokens": _log(rng, 16, 1024), "adapter": adapter, "kv": ""}
    return {"kind": kind, "shape": "7b", "layers": 2, "tokens": _log(rng, 32, 1500), "adapter": adapter, "kv": ""}


# ---- models -------------------------------------------------------------------------------------

def _shape(case):
    import dataclasses
    s = I.SHAPES[case["shape"]]
    return dataclasses.replace(s, n_layers=case["layers"], kv=case["kv"] or s.kv, adapter=case["adapter"])


def _gen(seed, *key):
    h = seed & 0xFFFFFFFF
    for k in key:
        h = (h * 1000003 + int(k) + 17) & 0x7FFFFFFFFFFF
    return torch.Generator(device="cuda").manual_seed(h)


def _randn(seed, key, rows, cols, scale, dt):
    g = _gen(seed, *key)
    return (torch.randn(rows, cols, generator=g, device="cuda", dtype=torch.float32) * scale).to(dt)


class Weights:
    """The tensors of a seed's model, made again on each request: (kind, layer) -> device tensor in the storage type."""

    def __init__(self, shape, seed, weak=0.0):
        self.s, self.seed = shape, seed
        self.dt = torch.float32 if shape.dtype == "f32" else torch.bfloat16
        V, d = shape.vocab, shape.d_model
        self.next = torch.randperm(V, generator=_gen(seed, 901), device="cuda")
        is_weak = torch.rand(V, generator=_gen(seed, 902), device="cuda") < weak
        self.row_scale = torch.where(is_weak, 0.36 * math.sqrt(4096 / d) if d >= 2048 else 0.3 if d >= 512 else 0.36, 1.0)
        self.rows = {(k, l): (r, c) for k, l, r, c in I.tensor_list(shape)}

    def get(self, kind, layer):
        r, c = self.rows[(kind, layer)]
        s = self.s
        if kind in (I.KIND_FINAL_NORM, I.KIND_NORM1, I.KIND_NORM2, I.KIND_A_NORM_IN, I.KIND_A_NORM_LAST, I.KIND_A_NORM_POST):
            return (1.0 + 0.1 * _randn(self.seed, (kind, layer + 1), 1, c, 1.0, torch.float32)).reshape(c).to(self.dt)
        if kind == I.KIND_EMBED:
            return _randn(self.seed, (kind, 0), r, c, 1.0, self.dt)
        if kind in (I.KIND_LM_HEAD, I.KIND_A_HEAD):
            e = self.get(I.KIND_EMBED, -1).float() * (self.row_scale * (1.28 / math.sqrt(s.d_model)))[:, None]
            out = torch.empty_like(e)
            out[self.next] = e
            return out.to(self.dt)
        scale = STD
        if (kind in (I.KIND_WO, I.KIND_WD) and layer >= s.exit_layer) or kind in (I.KIND_A_WO, I.KIND_A_WD, I.KIND_A_W2):
            scale = STD * ALPHA
        return _randn(self.seed, (kind, layer + 1), r, c, scale, self.dt)


def _load(shape, seed, max_seq, weak=0.0):
    kg = B.Kangaroo(shape, max_seq, gamma_max=GAMMA, kv_page_tokens=PAGE)
    kg.kv.zero_()
    w = Weights(shape, seed, weak)
    for kind, layer in w.rows:
        t = w.get(kind, layer)
        kg._chk(kg.L.kg_load_tensor(kg.h, kind, layer, t.data_ptr(), t.numel()))
    return kg, w


def _prompt(shape, seed, n):
    """Random token ids, the same on every machine."""
    return I.gen_prompt(shape.vocab, n, seed=(seed * 7919 + 13) & 0x7FFFFFFF)


def _continuation(w, last, n):
    """The n tokens the model prefers after token `last`."""
    nxt = w.next.cpu().numpy()
    out = []
    for _ in range(n):
        last = int(nxt[last])
        out.append(last)
    return out


# ---- one pass -----------------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        L, code = B.lib(), 1 if case["dtype"] == "bf16" else 0
        w, x = _linear_inputs(case, seed)
        packed = torch.empty(L.kg_op_packed_bytes(code, N, K), dtype=torch.uint8, device="cuda")
        work = torch.empty(L.kg_op_work_bytes(K), dtype=torch.uint8, device="cuda")
        y = torch.empty((M, N), dtype=torch.float32, device="cuda")
        stream = torch.cuda.current_stream().cuda_stream
        rc = L.kg_op_pack(code, w.data_ptr(), N, K, packed.data_ptr(), stream)
        if rc != 0:
            raise RuntimeError("kg_op_pack: %d" % rc)
        torch.cuda.synchronize()
        return {"kind": kind, "L": L, "keep": (x, packed, work), "y": y,
                "args": (code, packed.data_ptr(), N, K, x.data_ptr(), M, y.data_ptr(), work.data_ptr(), stream)}
    shape = _shape(case)
    T = case["tokens"]
    st = {"kind": kind}
    if kind in ("train", "features"):
        kg, _ = _load(shape, seed, T + 16, 1.0)                    # every distribution spread out, as a training set's are
        kg.train_bind(T)
        # the caller's workspace holds the parameter block first and the gradient block behind it (256-byte aligned)
        n = kg.train_param_count()
        off = (4 * n + 255) // 256 * 256
        st.update(kg=kg, grads=kg.train_work[off:off + 4 * n].view(torch.float32), tokens=_prompt(shape, seed, T))
        if kind == "features":
            st["F"], st["Zt"] = _features(shape, seed, T)
        return st
    new = case.get("new", 0)
    kg, w = _load(shape, seed, T + new + GAMMA + 2, case.get("weak", 0.0))
    st.update(kg=kg, prompt=_prompt(shape, seed, T), new=new)
    mode = case.get("mode", 0)
    st["params"], st["keep"] = B.make_params(mode=mode, temperature=1.0, eta=ETA, gamma=GAMMA, seed=seed)
    if kind == "prefill":
        es = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[shape.kv_dtype]
        n = _pages(T + GAMMA + 2) * (shape.n_layers + 1) * shape.n_heads * 2 * PAGE * shape.head_dim
        st["kv"] = kg.kv.view(es)[:n]
    if kind == "plain":
        st["forced"] = _continuation(w, int(st["prompt"][-1]), new)
    torch.cuda.synchronize()
    return st


def _pages(max_seq):
    return (max_seq + PAGE - 1) // PAGE


def _linear_inputs(case, seed):
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    return _randn(seed, (1, 1), case["N"], case["K"], STD, dt), _randn(seed, (1, 2), case["M"], case["K"], 1.0, torch.float32)


def _features(shape, seed, T):
    """Early features as large as a residual stream after the exit layer, and target logits with one token that stands out."""
    F = _randn(seed, (3, 1), T, shape.d_model, 2.5, torch.float32)
    Zt = _randn(seed, (3, 2), T, shape.vocab, 1.28, torch.float32)
    top = torch.randint(0, shape.vocab, (T, 1), generator=_gen(seed, 3, 3), device="cuda")
    Zt.scatter_(1, top, 12.0)
    return F, Zt


def run(st):
    kind = st["kind"]
    if kind == "linear":
        rc = st["L"].kg_op_linear(*st["args"])
        if rc != 0:
            raise RuntimeError("kg_op_linear: %d" % rc)
        return st["y"]
    kg = st["kg"]
    if kind == "train":
        return {"loss": kg.train_step(st["tokens"], lr=1e-5), "grads": st["grads"]}
    if kind == "features":
        loss = kg.train_accumulate_features(st["F"], st["Zt"])
        kg.train_apply(lr=1e-5)
        return {"loss": loss, "grads": st["grads"]}
    p = st["params"]
    if kind == "prefill":
        token = kg.prefill(p, st["prompt"])
        return {"token": token, "logits": kg.read_logits(1, 0), "kv": st["kv"]}
    if kind == "plain":
        tokens, logits = [kg.prefill(p, st["prompt"])], [kg.read_logits(1, 0)]
        for t in st["forced"]:
            tokens.append(kg.plain_step(p, t))
            logits.append(kg.read_logits(1, 0))
        return {"tokens": np.array(tokens), "logits": np.stack(logits)}
    tokens, _ = kg.generate(p, st["prompt"], st["new"])
    return {"tokens": np.array(tokens), "logits": kg.read_logits(1, 0)}


# ---- what a pass cannot do without --------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "linear":
        M, N, K, e = case["M"], case["N"], case["K"], 2 if case["dtype"] == "bf16" else 4
        return {"bytes": e * N * K + 4 * M * (N + K), "flops": 2 * M * N * K}
    s = _shape(case)
    d, f, V, L, l, T = s.d_model, s.d_ffn, s.vocab, s.n_layers, s.exit_layer, case["tokens"]
    e, ekv = s.bytes_per_weight(), {"f32": 4, "bf16": 2, "f16": 2}[s.kv_dtype]
    layer, attn_w, head = 4 * d * d + 3 * d * f, 4 * d * d, V * d
    a = case["adapter"]
    adapter = {0: attn_w, 1: attn_w, 2: layer, 3: 2 * d * d}[a]
    kv_pos = 2 * d * ekv                                         # one layer's cached keys and values of one position
    kv_slots = L + (0 if a == 3 else 1)
    a_kv_w = 0 if a == 3 else 2 * d * d                          # the prompt pass needs the adapter's keys and values only
    # prompt pass: every weight and the rows' embeddings read, the cache written; the head for one row
    pb = e * (L * layer + a_kv_w + head + T * d) + T * kv_slots * kv_pos + 4 * V
    pf = 2 * T * (L * layer + a_kv_w) + 2 * head + L * 2 * T * T * d
    if kind == "prefill":
        return {"bytes": pb, "flops": pf}
    new = case.get("new", 0)

    def forward(layers, rows, pos, extra):                       # a decode forward at position pos: bytes, flops
        w = layers * layer + extra
        return e * w + layers * pos * kv_pos + 4 * rows * V, 2 * rows * w + layers * 4 * rows * pos * d
    if kind == "plain":
        for i in range(new):
            b, fl = forward(L, 1, T + i, head)
            pb, pf = pb + b, pf + fl
        return {"bytes": pb, "flops": pf}
    if kind == "kangaroo":
        # k drafts a round (drafting stops at a weak token or at gamma), all accepted: k + 1 tokens
        q = 1.0 - case["weak"]
        k = sum(q ** i for i in range(GAMMA))
        rounds = max(1.0, (new - 1) / (k + 1))
        pos = T + new / 2
        b1, f1 = forward(l, 1, pos, adapter + head)
        b2, f2 = forward(l, 1, pos, 0)
        b3, f3 = forward(L - l, k + 1, pos, head)
        return {"bytes": pb + rounds * (k * (b1 + (0 if a == 3 else pos * kv_pos)) + b2 + b3), "flops": pf + rounds * (k * f1 + f2 + f3)}
    # training: adapter forward and the two backward products per weight, the head three times (target, draft, its input's gradient)
    own = head if a in (1, 3) else 0
    nparam = adapter + own
    at = 0 if a == 3 else 6 * T * T * d
    gf = 6 * T * adapter + (6 if own else 4) * T * head + at
    gb = 4 * nparam * 8 + (e * head if not own else 0) + e * nparam + 4 * T * (2 * V + d)   # P, G, two moments read and written
    if kind == "features":
        return {"bytes": gb, "flops": gf}
    return {"bytes": e * (L * layer + head) + gb, "flops": gf + 2 * T * (L * layer + head) + L * 2 * T * T * d}


def tolerance(case):
    """About four times the error against 64 bits that a pass was measured to have (in brackets)."""
    kind = case["kind"]
    if kind == "linear":
        return {"rel": 1e-5 if case["dtype"] == "bf16" else 2e-6}       # bf16: rows split in two bf16 parts, 2^-17 (2.5e-6)
    if kind == "features":
        return {"rel": 1.5e-5}                                          # float32 throughout (3.3e-6)
    if kind == "train":
        return {"rel": 2e-3}                                            # gradients behind the frozen model's 16-bit cache (3e-4 .. 4e-4)
    if case["shape"] == "toy":
        return {"rel": 1e-5}                                            # float32 throughout (1e-7 .. 3e-6)
    # the 16-bit caches round keys and values (2^-12 half, 2^-9 bfloat16), and a value near the middle may
    # round either way (3e-4 .. 9e-4 with the half cache, 2e-3 .. 3e-3 with the bfloat16 one)
    return {"rel": 0.012 if case["kv"] == "bf16" else 3e-3}


# ---- the same in 64 bits ------------------------------------------------------------------------

class Exact:
    """The model in float64, whole sequences at once, no cache and none of the framework's code."""

    def __init__(self, shape, seed, weak=0.0):
        self.s, self.w = shape, Weights(shape, seed, weak)

    def t(self, kind, layer=-1):
        return self.w.get(kind, layer).double()

    def norm(self, x, g):
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + self.s.rms_eps) * g

    def rope(self, x):                                            # [T][H][hd]
        T, hd = x.shape[0], self.s.head_dim
        inv = self.s.rope_theta ** (-2.0 * torch.arange(hd // 2, device="cuda", dtype=torch.float64) / hd)
        a = torch.arange(T, device="cuda", dtype=torch.float64)[:, None] * inv
        c, s = a.cos()[:, None], a.sin()[:, None]
        x0, x1 = x[..., : hd // 2], x[..., hd // 2:]
        return torch.cat([x0 * c - x1 * s, x1 * c + x0 * s], -1)

    def attention(self, n, wq, wk, wv, keep=None):
        T, H, hd = n.shape[0], self.s.n_heads, self.s.head_dim
        q, k, v = ((n @ w.T).reshape(T, H, hd) for w in (wq, wk, wv))
        q, k = self.rope(q), self.rope(k)
        if keep is not None:
            keep.append((k, v))
        mask = torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1)
        out = []
        for h in range(H):
            sc = (q[:, h] @ k[:, h].T / math.sqrt(hd)).masked_fill(mask, -math.inf)
            out.append(torch.softmax(sc, -1) @ v[:, h])
        return torch.cat(out, -1)

    def block(self, x, i, keep=None):
        t = self.t
        n = self.norm(x, t(I.KIND_NORM1, i))
        x = x + self.attention(n, t(I.KIND_WQ, i), t(I.KIND_WK, i), t(I.KIND_WV, i), keep) @ t(I.KIND_WO, i).T
        n = self.norm(x, t(I.KIND_NORM2, i))
        return x + (torch.nn.functional.silu(n @ t(I.KIND_WG, i).T) * (n @ t(I.KIND_WU, i).T)) @ t(I.KIND_WD, i).T

    def layers(self, tokens, keep=None):
        """(early features, last hidden states) of every position."""
        x = self.w.get(I.KIND_EMBED, -1)[torch.as_tensor(np.asarray(tokens), device="cuda").long()].double()
        early = None
        for i in range(self.s.n_layers):
            x = self.block(x, i, keep)
            if i == self.s.exit_layer - 1:
                early = x
        return early, x

    def target(self, x):
        return self.norm(x, self.t(I.KIND_FINAL_NORM)) @ self.t(I.KIND_LM_HEAD).T

    def adapter_params(self):
        a = self.s.adapter
        kinds = [I.KIND_A_W1, I.KIND_A_W2] if a == 3 else [I.KIND_A_WQ, I.KIND_A_WK, I.KIND_A_WV, I.KIND_A_WO]
        kinds += [I.KIND_A_NORM_IN, I.KIND_A_NORM_LAST]
        kinds += [I.KIND_A_HEAD] if a in (1, 3) else []
        kinds += [I.KIND_A_NORM_POST, I.KIND_A_WG, I.KIND_A_WU, I.KIND_A_WD] if a == 2 else []
        return {k: self.t(k) for k in kinds}

    def draft(self, F, p):
        """Draft logits of every position from the early features."""
        a, silu = self.s.adapter, torch.nn.functional.silu
        n = self.norm(F, p[I.KIND_A_NORM_IN])
        if a == 3:
            h = F + silu(n @ p[I.KIND_A_W1].T) @ p[I.KIND_A_W2].T
        else:
            h = F + self.attention(n, p[I.KIND_A_WQ], p[I.KIND_A_WK], p[I.KIND_A_WV]) @ p[I.KIND_A_WO].T
        if a == 2:
            b = self.norm(h, p[I.KIND_A_NORM_POST])
            h = h + (silu(b @ p[I.KIND_A_WG].T) * (b @ p[I.KIND_A_WU].T)) @ p[I.KIND_A_WD].T
        head = p[I.KIND_A_HEAD] if a in (1, 3) else self.t(I.KIND_LM_HEAD)
        return self.norm(h, p[I.KIND_A_NORM_LAST]) @ head.T


def exact(case, seed):
    kind = case["kind"]
    if kind == "linear":
        w, x = _linear_inputs(case, seed)
        return x.double() @ w.double().T
    shape = _shape(case)
    T, new = case["tokens"], case.get("new", 0)
    m = Exact(shape, seed, 1.0 if kind in ("train", "features") else case.get("weak", 0.0))
    if kind in ("train", "features"):
        if kind == "train":
            with torch.no_grad():
                F, x = m.layers(_prompt(shape, seed, T))
                Zt = m.target(x)
        else:
            F, Zt = (v.double() for v in _features(shape, seed, T))
        p = {k: v.requires_grad_() for k, v in m.adapter_params().items()}
        loss = -(torch.softmax(Zt, -1) * torch.log_softmax(m.draft(F, p), -1)).sum()
        grads = torch.autograd.grad(loss, list(p.values()))
        return {"loss": float(loss.detach()), "grads": torch.cat([g.reshape(-1) for g in grads])}
    with torch.no_grad():
        prompt = _prompt(shape, seed, T)
        if kind == "prefill":
            cache = []
            early, x = m.layers(prompt, cache)
            if shape.adapter != 3:
                p = m.adapter_params()
                n = m.norm(early, p[I.KIND_A_NORM_IN])
                H, hd = shape.n_heads, shape.head_dim
                k, v = ((n @ p[i].T).reshape(T, H, hd) for i in (I.KIND_A_WK, I.KIND_A_WV))
                cache.append((m.rope(k), v))
            # pool: [page][cache][head][keys, values][position][dimension]
            n_pages = _pages(T + GAMMA + 2)
            pool = torch.zeros(n_pages, shape.n_layers + 1, shape.n_heads, 2, PAGE, shape.head_dim, dtype=torch.float64, device="cuda")
            for slot, kv in enumerate(cache):
                for j, c in enumerate(kv):
                    for pg in range((T + PAGE - 1) // PAGE):
                        part = c[pg * PAGE:(pg + 1) * PAGE]
                        pool[pg, slot, :, j, : part.shape[0]] = part.transpose(0, 1)
            return {"token": None, "logits": m.target(x[-1:])[0], "kv": pool.reshape(-1)}
        chain = _continuation(m.w, int(prompt[-1]), new + GAMMA + 1)
        if kind == "plain":
            _, x = m.layers(list(prompt) + chain[:new])
            return {"tokens": None, "logits": m.target(x[T - 1:T + new])}
        # Kangaroo: the request follows the chain of preferred tokens; the rounds follow from the drafts' confidences, and
        # what is compared is the target's first row of the last round, at the position of that round's pending token
        early, x = m.layers(list(prompt) + chain)
        conf = torch.softmax(m.draft(early, m.adapter_params()), -1).amax(-1).cpu().numpy()
        base, n = T, 1
        while n < new:
            k, row = 0, base
            while k < GAMMA:
                k += 1
                if conf[base + k - 1] < ETA:
                    break
            base, n = base + k + 1, n + k + 1
        return {"tokens": None, "logits": m.target(x[row:row + 1])[0]}
