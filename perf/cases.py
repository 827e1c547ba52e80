"""Performance cases: the calls a program makes of this library, timed and
checked one pass at a time.

A decoder round with this library is: prefill a prompt once, then per round
draft a tree (dv_draft_forward over the tree so far), verify it with the target
(dv_verify_step), pick the accepted path (greedily inside the step, or with
dv_accept_sampled at temperature > 0) and commit it (dv_kv_commit).  The listed
cases are those calls on the shapes of the benchmark and the tests: the tiny
model, Llama-7B/13B-shaped layers and one whole 13B model.  Most models here
have a few layers only, so a case is the decoder layers plus the head; every
layer of a model is the same work.  draw() gives more of the same ranges: other
widths, head sizes, tree sizes, context and prompt lengths, weight types.

Inputs are random with the distributions of the synthetic workloads: weights
N(0, 0.02^2), gains 1 + N(0, 0.1^2), committed keys and values N(0, 0.02^2 d).
"""
import ctypes
import math

import numpy as np
import torch

from paper_2412_18934_amd import dv
from paper_2412_18934_amd.device import LAYER_KEYS, MATRIX_KEYS, make_config

EPS, ROPE_BASE, STD = 1e-6, 10000.0, 0.02
TINY = dict(d_model=256, n_heads=4, d_ffn=688, vocab=1024)
SEVEN = dict(d_model=4096, n_heads=32, d_ffn=11008, vocab=32000)
THIRTEEN = dict(d_model=5120, n_heads=40, d_ffn=13824, vocab=32000)


def listed():
    return [
        # the smallest model: launches and latency are all there is
        dict(name="tiny-f32-chain4", kind="verify", dtype="f32", n_layers=2, **TINY, ctx=64, n_tree=4, depth=4,
             commit=False),
        # one decoding round of a 7B-shaped target: verify 8 nodes, commit the deepest branch
        dict(name="7b-round-m8-ctx512", kind="verify", dtype="bf16", n_layers=4, **SEVEN, ctx=512, n_tree=8, depth=5,
             commit=True),
        # the headline: a whole 13B-shaped model verifies 16 nodes
        dict(name="13b-verify-m16-ctx1024", kind="verify", dtype="bf16", n_layers=40, **THIRTEEN, ctx=1024, n_tree=16,
             depth=6, commit=False),
        # the paper's large candidate count (60 nodes) at a ragged context
        dict(name="13b-verify-m60-ctx777", kind="verify", dtype="bf16", n_layers=4, **THIRTEEN, ctx=777, n_tree=60,
             depth=8, commit=False),
        # a long conversation: the cache is a large part of the bytes
        dict(name="13b-verify-m16-ctx8192", kind="verify", dtype="bf16", n_layers=3, **THIRTEEN, ctx=8192, n_tree=16,
             depth=6, commit=False),
        # the paper's int8 target
        dict(name="13b-int8-verify-m16-ctx1024", kind="verify", dtype="i8", n_layers=4, **THIRTEEN, ctx=1024,
             n_tree=16, depth=6, commit=False),
        # the paper's float32 target (its server setting)
        dict(name="7b-f32-verify-m16-ctx512", kind="verify", dtype="f32", n_layers=2, **SEVEN, ctx=512, n_tree=16,
             depth=6, commit=False),
        # a long prompt
        dict(name="13b-prefill-1024", kind="prefill", dtype="bf16", n_layers=4, **THIRTEEN, ctx=0, n_prompt=1024),
        # a chat turn: a short prompt behind a cached conversation
        dict(name="7b-prefill-150-ctx333", kind="prefill", dtype="bf16", n_layers=4, **SEVEN, ctx=333, n_prompt=150),
        # a prompt of medium length on the int8 target
        dict(name="13b-int8-prefill-500", kind="prefill", dtype="i8", n_layers=2, **THIRTEEN, ctx=0, n_prompt=500),
        # one pass of a one-block draft while its tree is grown
        dict(name="13b-draft-pass-m10", kind="draft", dtype="bf16", n_layers=1, **THIRTEEN, ctx=1024, n_tree=10,
             depth=4),
        # the sampling rule at T = 1 over 16 nodes' logits
        dict(name="accept-sampled-m16", kind="sample", dtype="bf16", n_layers=1, d_model=256, n_heads=4, d_ffn=688,
             vocab=32000, n_tree=16, depth=6, temperature=1.0),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_model(rng, dtype):
    """A Llama-shaped model: the two named shapes or a width in between, FFN
    about 2.7 times the width."""
    shape = rng.random()
    if shape < 0.25:
        m = dict(SEVEN)
    elif shape < 0.5:
        m = dict(THIRTEEN)
    else:
        hd = rng.choice([64, 128])
        d = 256 * _log_int(rng, 1, 20)
        m = dict(d_model=d, n_heads=d // hd, d_ffn=64 * max(1, round(d * rng.uniform(2.5, 3.2) / 64)), vocab=32000)
    if rng.random() < 0.4:
        m["vocab"] = 32 * _log_int(rng, 32, 1000)
    m["n_layers"] = rng.randint(1, 2 if dtype == "f32" else 3)
    m["dtype"] = dtype
    return m


def draw(rng):
    kind = rng.choices(["verify", "prefill", "draft", "sample"], [6, 4, 1.5, 1])[0]
    dtype = "bf16" if kind in ("draft", "sample") else rng.choices(["bf16", "i8", "f32"], [5, 3, 2])[0]
    c = dict(kind=kind, **_draw_model(rng, dtype))
    if kind == "prefill":
        c["ctx"] = 0 if rng.random() < 0.5 else _log_int(rng, 8, 2048)
        # float32 prompts are short here: the type is for small models
        c["n_prompt"] = _log_int(rng, 16, 200 if dtype == "f32" else 1500 if dtype == "bf16" else 1100)
        return c
    c["n_tree"] = _log_int(rng, 1, 64)
    c["depth"] = rng.randint(2, 9) if c["n_tree"] > 1 else 1
    if kind == "sample":
        c.update(n_layers=1, d_model=256, n_heads=4, d_ffn=688, temperature=rng.choice([0.6, 0.8, 1.0, 1.3]))
        return c
    c["ctx"] = rng.randint(1, 40) if rng.random() < 0.1 else _log_int(rng, 32, 8192)
    if kind == "verify":
        c["commit"] = rng.random() < 0.5
    else:
        c["n_layers"] = rng.randint(1, 2)
    return c


# ---------------------------------------------------------------------------
# inputs


class _Inputs:
    """Everything random of a case, made on the GPU from the seed."""

    def __init__(self, case, seed):
        self.c = c = case
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        host = np.random.default_rng(seed)
        d, f, v, i8 = c["d_model"], c["d_ffn"], c["vocab"], c["dtype"] == "i8"
        self.dense = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
        self.hd = d // c["n_heads"]
        self.layers = []
        shapes = dict(wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), w_gate=(f, d), w_up=(f, d), w_down=(d, f))
        for _ in range(c["n_layers"]):
            lay = {k: self._gain(d) for k in LAYER_KEYS if k not in MATRIX_KEYS}
            for k in MATRIX_KEYS:
                lay[k], lay[k + "_scale"] = self._matrix(shapes[k], i8)
            self.layers.append(lay)
        self.embed = self._normal((v, d), STD)
        self.final_norm = self._gain(d)
        self.lm_head, self.lm_scale = self._matrix((v, d), i8)
        if c["kind"] == "draft":
            self.dgf = [self._normal((d, k), STD) for k in (d, d, 2 * d)]
            self.feat = self._normal((c["n_tree"], d), 1.0).float()
        if c["kind"] == "prefill":
            self.tokens = host.integers(0, v, c["n_prompt"]).astype(np.int32)
        else:
            self.tokens, self.parents = _tree(host, c["n_tree"], c["depth"], v, c["kind"] == "verify" and
                                              c["depth"] == c["n_tree"])
        if c["kind"] == "sample":
            self._sample_inputs(host)

    def _normal(self, shape, std, dtype=None):
        t = torch.empty(shape, dtype=dtype or self.dense, device="cuda")
        return t.normal_(0.0, std, generator=self.g)

    def _gain(self, n):
        return self._normal((n,), 0.1).add_(1.0)

    def _matrix(self, shape, i8):
        if not i8:
            return self._normal(shape, STD), None
        code = torch.empty(shape, dtype=torch.int8, device="cuda")
        step = max(1, (1 << 26) // shape[1])
        for r in range(0, shape[0], step):
            part = self._normal((min(step, shape[0] - r), shape[1]), 127 / 4, torch.float32)
            code[r:r + step] = part.round_().clamp_(-127, 127).to(torch.int8)
        scale = torch.empty(shape[0], device="cuda").uniform_(0.75, 1.25, generator=self.g).mul_(STD * 4 / 127)
        return code, scale

    def cache(self, capacity):
        """K [L][H][cap][hd] and V [L][H][cap/32][hd][32], ctx slots committed."""
        c = self.c
        shape = (c["n_layers"], c["n_heads"], capacity, self.hd)
        std = STD * math.sqrt(c["d_model"])
        k, v = self._normal(shape, std), self._normal(shape, std)
        k[:, :, c["ctx"]:] = 0
        v[:, :, c["ctx"]:] = 0
        return k, _v_tiles(v)

    def _sample_inputs(self, host):
        # the target's logits, and a draft that resembles it; children are
        # drawn from the draft's distribution at their parent
        c = self.c
        n, v = c["n_tree"], c["vocab"]
        self.logits = self._normal((n, v), 3.0, torch.float32)
        noise = self._normal((n, v), 0.7, torch.float32)
        self.q = torch.softmax((self.logits + noise) / c["temperature"], dim=1).contiguous()
        pick = torch.multinomial(self.q, n, replacement=True, generator=self.g).cpu().numpy()
        for i in range(1, n):
            self.tokens[i] = pick[self.parents[i], i]
        self.u_accept = host.random(n, dtype=np.float32)
        self.u_bonus = host.random(n, dtype=np.float32)


def _tree(host, n, depth, vocab, chain):
    parents, dep = np.full(n, -1, np.int32), np.ones(n, np.int64)
    for i in range(1, n):
        ok = [j for j in range(i) if dep[j] < depth]
        parents[i] = i - 1 if chain else ok[int(host.integers(len(ok)))]
        dep[i] = dep[parents[i]] + 1
    return host.integers(0, vocab, n).astype(np.int32), parents


def _path(parents):
    """The root-to-node path of the deepest node (the first of them)."""
    depth = []
    for p in parents:
        depth.append(1 if p < 0 else depth[p] + 1)
    node, path = int(np.argmax(depth)), []
    while node >= 0:
        path.append(node)
        node = int(parents[node])
    return path[::-1]


def _v_tiles(v):
    n_l, n_h, cap, hd = v.shape
    return v.view(n_l, n_h, cap // 32, 32, hd).transpose(3, 4).contiguous()


# ---------------------------------------------------------------------------
# the calls


class _State:
    """What a program keeps: weights, handle, cache, output buffers."""

    def __init__(self, case, seed):
        self.h = None
        self.c = c = case
        self.i = i = _Inputs(case, seed)
        if c["kind"] == "sample":
            c = dict(c, ctx=0)
        n = c.get("n_prompt", c.get("n_tree"))
        capacity = -(-(c["ctx"] + n) // 32) * 32
        cfg = make_config(c["n_layers"], c["d_model"], c["n_heads"], i.hd, c["d_ffn"], c["vocab"], EPS, ROPE_BASE,
                          c["dtype"], max(capacity, 64), 64)
        pp = ctypes.POINTER(ctypes.c_void_p)
        self.tables = {k: (ctypes.c_void_p * c["n_layers"])(*[lay[k].data_ptr() for lay in i.layers])
                       for k in i.layers[0] if i.layers[0][k] is not None}
        table = {k: ctypes.cast(t, pp) for k, t in self.tables.items()}
        self.w = dv.dv_weights(i.embed.data_ptr(), i.final_norm.data_ptr(), i.lm_head.data_ptr(),
                               *[table[k] for k in LAYER_KEYS],
                               None if i.lm_scale is None else i.lm_scale.data_ptr(),
                               *[table.get(k + "_scale") for k in MATRIX_KEYS])
        if c["kind"] == "draft":
            self.dgf = dv.dv_dgf_weights(*[t.data_ptr() for t in i.dgf])
            self.h = dv.dv_draft_init(cfg, self.w, self.dgf)
            self.feat_out = torch.empty((n, c["d_model"]), dtype=torch.float32, device="cuda")
        else:
            self.h = dv.dv_verify_init(cfg, self.w)
        if c["kind"] in ("verify", "draft"):
            self.logits = torch.empty((n, c["vocab"]), dtype=torch.float32, device="cuda")
        if c["kind"] != "sample":
            self.k, self.v = i.cache(capacity)
            self.kv = dv.dv_kv(self.k.data_ptr(), self.v.data_ptr(), capacity, c["ctx"])
        if c["kind"] == "verify":
            self.path = _path(i.parents)
        torch.cuda.synchronize()

    def __del__(self):
        if self.h is not None:
            dv.dv_verify_free(self.h)


def prepare(case, seed):
    return _State(case, seed)


def run(s):
    c, i = s.c, s.i
    if c["kind"] == "sample":
        acc = dv.dv_accept_sampled(s.h, s.i.logits.data_ptr(), i.tokens, i.parents, i.q.data_ptr(), c["temperature"],
                                   i.u_accept, i.u_bonus)
        return {"accept": np.frombuffer(acc, np.int32)}
    s.kv.len = c["ctx"]
    if c["kind"] == "prefill":
        token = dv.dv_prefill(s.h, i.tokens, s.kv)
        return {"k": s.k, "v": s.v, "next": token}
    if c["kind"] == "draft":
        dv.dv_draft_forward(s.h, i.tokens, i.parents, s.kv, i.feat.data_ptr(), s.feat_out.data_ptr(),
                            s.logits.data_ptr())
        return {"logits": s.logits, "features": s.feat_out, "k": s.k, "v": s.v}
    acc = dv.dv_verify_step(s.h, i.tokens, i.parents, s.kv, s.logits.data_ptr())
    out = {"logits": s.logits, "accept": np.frombuffer(acc, np.int32), "k": s.k, "v": s.v}
    if c["commit"]:
        # the caller's own acceptance rule took the deepest branch
        own = dv.dv_accept.from_buffer_copy(acc)
        own.accept_len = len(s.path)
        own.path[:len(s.path)] = s.path
        dv.dv_kv_commit(s.h, s.kv, own)
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without


def work(case):
    c = case
    d, f, v = c["d_model"], c["d_ffn"], c["vocab"]
    if c["kind"] == "sample":
        # at least the root's two rows are read (the walk's length is random)
        return {"bytes": 2 * 4 * v, "flops": 8 * v}
    size = {"bf16": 2, "i8": 1, "f32": 4}[c["dtype"]]
    kv = 4 if c["dtype"] == "f32" else 2
    n = c.get("n_prompt", c.get("n_tree"))
    params = c["n_layers"] * (4 * d * d + 3 * d * f)
    head = v * d
    if c["kind"] == "draft":
        params += 4 * d * d
    keys = c["n_layers"] * 2 * d * kv
    read = c["ctx"] * keys + n * d * kv
    write = n * keys + (4 * n * v if c["kind"] != "prefill" else 4)
    if c["kind"] == "prefill":
        attended = n * c["ctx"] + n * (n + 1) // 2
        head_rows = 1
    else:
        attended = n * c["ctx"] + n * c["depth"]
        head_rows = n
    return {"bytes": (params + head) * size + read + write,
            "flops": 2 * n * params + 2 * head_rows * head + 4 * c["n_layers"] * d * attended}


def tolerance(case):
    c = case
    if c["kind"] == "sample":
        return {"rel": 0.0, "differ": 0.009}  # one of the struct's words: a draw at a boundary of the CDF
    if c["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.009}
    # new keys and values are rounded to bf16: one that lands on the other
    # side of a midpoint is off by up to 2^-7 of itself and goes on into the
    # layers above, the more the more of the attended rows are new (measured
    # against 64 bits: 1e-4 for trees, 9e-4 for a 1024-token prompt)
    return {"rel": 4e-3 if c["kind"] == "prefill" else 5e-4, "max": 0.05, "differ": 0.009}


# ---------------------------------------------------------------------------
# the same in 64 bits


def _w64(lay, k):
    w = lay[k].double()
    s = lay.get(k + "_scale")
    return w if s is None else w.mul_(s.double()[:, None])


def _norm64(x, gain):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gain.double()


def _rope64(x, pos, hd):
    # x [n][H][hd]; pairs (j, j + hd/2)
    theta = ROPE_BASE ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device="cuda") / hd)
    ang = pos.double()[:, None] * theta
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., :hd // 2], x[..., hd // 2:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _stack64(i, c, x, k, v, pos, mask):
    """Layers over rows x [n][d]; k, v [L][H][cap][hd] (64 bits) get the new
    rows at [ctx, ctx + n), rounded to the cache type; mask [n][ctx + n]."""
    n, hd, n_h, p = x.shape[0], i.hd, c["n_heads"], c["ctx"]
    bias = torch.zeros_like(mask, dtype=torch.float64).masked_fill_(~mask, -math.inf)
    for l, lay in enumerate(i.layers):
        u = _norm64(x, lay["attn_norm"])
        q = _rope64((u @ _w64(lay, "wq").T).view(n, n_h, hd), pos, hd)
        kn = _rope64((u @ _w64(lay, "wk").T).view(n, n_h, hd), pos, hd)
        vn = (u @ _w64(lay, "wv").T).view(n, n_h, hd)
        k[l, :, p:p + n] = kn.transpose(0, 1).to(i.dense).double()
        v[l, :, p:p + n] = vn.transpose(0, 1).to(i.dense).double()
        o = torch.empty(n_h, n, hd, dtype=torch.float64, device="cuda")
        for h in range(n_h):
            s = torch.softmax(q[:, h] @ k[l, h, :p + n].T / math.sqrt(hd) + bias, -1)
            o[h] = s @ v[l, h, :p + n]
        x = x + o.transpose(0, 1).reshape(n, -1) @ _w64(lay, "wo").T
        u = _norm64(x, lay["ffn_norm"])
        g = u @ _w64(lay, "w_gate").T
        x = x + (torch.nn.functional.silu(g) * (u @ _w64(lay, "w_up").T)) @ _w64(lay, "w_down").T
    return x


def exact(case, seed):
    c = case
    if c["kind"] == "sample":
        return None  # token ids and node numbers only
    i = _Inputs(c, seed)
    n = c.get("n_prompt", c.get("n_tree"))
    p = c["ctx"]
    capacity = -(-(p + n) // 32) * 32
    k, vt = i.cache(capacity)
    k, v = k.double(), vt.double().transpose(3, 4).reshape(k.shape).contiguous()
    tokens = torch.from_numpy(i.tokens).cuda().long()
    x = i.embed[tokens].double()
    mask = torch.ones(n, p + n, dtype=torch.bool, device="cuda")
    if c["kind"] == "prefill":
        pos = p + torch.arange(n, device="cuda")
        mask[:, p:] = torch.tril(mask[:, p:])
        _stack64(i, c, x, k, v, pos, mask)
        return {"k": k, "v": _v_tiles(v), "next": None}
    anc, dep = np.zeros((n, n), bool), np.ones(n, np.int64)
    for a in range(n):
        if i.parents[a] >= 0:
            anc[a] = anc[i.parents[a]]
            dep[a] = dep[i.parents[a]] + 1
        anc[a, a] = True
    mask[:, p:] = torch.from_numpy(anc).cuda()
    pos = p + torch.from_numpy(dep).cuda() - 1
    if c["kind"] == "draft":
        h1 = i.feat.double() @ i.dgf[0].double().T
        h2 = x @ i.dgf[1].double().T
        gate = torch.sigmoid(torch.cat([h1, h2], -1) @ i.dgf[2].double().T)
        x = gate * h1 + (1 - gate) * h2
    x = _stack64(i, c, x, k, v, pos, mask)
    logits = _norm64(x, i.final_norm) @ _w64({"w": i.lm_head, "w_scale": i.lm_scale}, "w").T
    if c["kind"] == "draft":
        return {"logits": logits, "features": x, "k": k, "v": _v_tiles(v)}
    if c["commit"]:
        at = p + torch.tensor(_path(i.parents), device="cuda")
        for t in (k, v):
            t[:, :, p:p + len(at)] = t[:, :, at].clone()
    return {"logits": logits, "accept": None, "k": k, "v": _v_tiles(v)}
