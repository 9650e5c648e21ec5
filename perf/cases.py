"""The work whose time this repository is tuned for: the calls a serving engine makes on one pipeline stage.

A stage is a slice of Llama-style decoder layers on one GPU.  An engine prefills packed prompts, runs decode steps of
one token per request against a paged KV cache, turns hidden states into tokens behind the last stage, and now and
then moves a request's cache between its pages and a packed buffer.  Every case is one such call (one is the chain of
calls that makes a token) through `paper_2506_10470_amd.tdp`.  Single layers stand for the stage they are part of: a
stage repeats the same kernels layer after layer, so a case holds one or two layers of a shape at its full width.

Shapes are the ones the repository's benchmark and tests use; contexts and prompts follow the log-normal lengths of
the benchmark's request mixes.
"""
import hashlib
import math

import numpy as np
import torch

from paper_2506_10470_amd import tdp

PAGE = 16

# name: (d_model, query heads, KV heads, head_dim, d_ff, q/k/v biases, rms_eps, rope_base,
#        (median, sigma, most) of the contexts, the same of the prompts)
SHAPES = {
    "tiny_gqa": (256, 8, 2, 64, 688, False, 1e-5, 1e4, (32, 0.5, 64), (16, 0.5, 32)),
    "tiny_bias": (320, 10, 2, 64, 688, True, 1e-6, 1e6, (32, 0.5, 64), (16, 0.5, 32)),
    "7b": (4096, 32, 32, 128, 11008, False, 1e-5, 1e4, (430, 0.7, 2560), (256, 0.8, 2048)),
    "13b": (5120, 40, 40, 128, 13824, False, 1e-5, 1e4, (830, 0.5, 4096), (384, 0.7, 4096)),
    "qwen32b": (5120, 40, 8, 128, 27648, True, 1e-6, 1e6, (830, 0.5, 4096), (384, 0.7, 4096)),
    "70b": (8192, 64, 8, 128, 28672, False, 1e-5, 1e4, (1024, 0.6, 4096), (1024, 0.6, 4096)),
}
K_SCALE, V_SCALE = 0.03125, 0.015625  # of the 8-bit caches


def listed():
    return [
        # the smallest calls: a two-layer toy stage, four requests - launches and their gaps are all there is
        {"name": "decode_tiny_b4", "kind": "decode", "shape": "tiny_gqa", "layers": 2, "n": 4, "kv8": False, "lens": 1},
        # few requests on a large model: the weights are streamed for 16 rows
        {"name": "decode_70b_b16", "kind": "decode", "shape": "70b", "layers": 2, "n": 16, "kv8": False, "lens": 2},
        # an ordinary batch that fits no tile: between the sizes that kernels are tuned at
        {"name": "decode_70b_b200", "kind": "decode", "shape": "70b", "layers": 2, "n": 200, "kv8": False, "lens": 3},
        # the benchmark's batch: the projections near the compute bound, attention the longest cache read
        {"name": "decode_70b_b512", "kind": "decode", "shape": "70b", "layers": 2, "n": 512, "kv8": False, "lens": 4},
        # the 8-bit cache in a large batch
        {"name": "decode_70b_b384_kv8", "kind": "decode", "shape": "70b", "layers": 2, "n": 384, "kv8": True, "lens": 5},
        # multi-head attention (one query head per KV head): the cache read outweighs everything
        {"name": "decode_13b_b128", "kind": "decode", "shape": "13b", "layers": 2, "n": 128, "kv8": False, "lens": 6},
        # one short prompt alone, as it arrives in an idle system
        {"name": "prefill_7b_p1", "kind": "prefill", "shape": "7b", "layers": 2, "n": 1, "kv8": False, "lens": 25},
        # a handful of ragged prompts, five query heads per KV head, biases
        {"name": "prefill_qwen32b_p8", "kind": "prefill", "shape": "qwen32b", "layers": 1, "n": 8, "kv8": False, "lens": 8},
        # the benchmark's prefill batch: the largest call
        {"name": "prefill_70b_p16", "kind": "prefill", "shape": "70b", "layers": 1, "n": 16, "kv8": False, "lens": 9},
        # behind the last stage: final norm, vocabulary projection, greedy token of a decode batch
        {"name": "lm_head_70b_b512", "kind": "head", "shape": "70b", "n": 512, "vocab": 32000},
        # moving requests without recomputing them: one group's cache goes into pages, another's comes out
        {"name": "kv_move_13b_s24", "kind": "move", "shape": "13b", "layers": 1, "n": 24, "kv8": False, "lens": 10},
        # the whole step from token ids to token ids: embedding, layers, head
        {"name": "token_step_7b_b48", "kind": "step", "shape": "7b", "layers": 4, "n": 48, "vocab": 32000, "kv8": False,
         "lens": 11},
    ]


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "head", "move", "step"])
    shape = rng.choice(["tiny_gqa", "tiny_bias", "7b", "13b", "qwen32b", "70b", "70b"])
    seed = rng.randrange(1000, 1 << 30)

    def spread(lo, hi):  # uniform in the logarithm, odd sizes as often as even ones
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))

    if kind == "decode":
        return {"kind": kind, "shape": shape, "layers": rng.choice([1, 2]), "n": spread(1, 256 if shape == "13b" else 512),
                "kv8": rng.random() < 0.25, "lens": seed}
    if kind == "prefill":
        return {"kind": kind, "shape": shape, "layers": 1, "n": spread(1, 8 if shape == "70b" else 24),
                "kv8": rng.random() < 0.25, "lens": seed}
    if kind == "head":
        return {"kind": kind, "shape": shape, "n": spread(1, 512), "vocab": rng.choice([1000, 8004, 32000])}
    if kind == "move":
        return {"kind": kind, "shape": shape, "layers": 1, "n": spread(1, 32), "kv8": rng.random() < 0.25, "lens": seed}
    return {"kind": kind, "shape": shape, "layers": rng.choice([1, 2]), "n": spread(1, 128), "vocab": rng.choice([1000, 32000]),
            "kv8": rng.random() < 0.25, "lens": seed}


# ---- what a case consists of ------------------------------------------------------------------------------------

class Dims:
    def __init__(self, case):
        (self.d, self.hq, self.hkv, self.dh, self.ff, self.bias, self.eps, self.base, self.ctx, self.prompt) = SHAPES[case["shape"]]
        self.layers = case.get("layers", 0)
        self.dq, self.dkv = self.hq * self.dh, self.hkv * self.dh
        self.params = self.d * (2 * self.dq + 2 * self.dkv) + 3 * self.d * self.ff  # of one layer


def lengths(case):
    """Tokens of every request: cached before the call (decode, step, move) or in the prompt (prefill)."""
    D = Dims(case)
    median, sigma, most = D.prompt if case["kind"] == "prefill" else D.ctx
    z = np.random.RandomState(case["lens"]).standard_normal(2 * case["n"] if case["kind"] == "move" else case["n"])
    return np.clip(np.rint(median * np.exp(sigma * z)), 4, most).astype(np.int64)


def number(seed, *what):
    return int.from_bytes(hashlib.blake2b(repr((int(seed),) + what).encode(), digest_size=7).digest(), "big")


def normal(seed, what, shape, std=1.0, mean=0.0, dtype=torch.bfloat16):
    g = torch.Generator(device="cuda").manual_seed(number(seed, what))
    x = torch.randn(shape, generator=g, device="cuda", dtype=dtype)
    if std != 1.0:
        x *= std
    return x + mean if mean else x


def layer_weights(D, seed, l):
    """The matrices of one layer [in, out] ~ N(0, 0.02), gains around 1, biases ~ N(0, 0.5)."""
    sizes = {"wq": (D.d, D.dq), "wk": (D.d, D.dkv), "wv": (D.d, D.dkv), "wo": (D.dq, D.d), "wg": (D.d, D.ff),
             "wu": (D.d, D.ff), "wd": (D.ff, D.d)}
    for name, shape in sizes.items():
        yield name, normal(seed, (l, name), shape, 0.02)
    for name in ("g_attn", "g_mlp"):
        yield name, normal(seed, (l, name), (D.d,), 0.02, 1.0, torch.float32)
    if D.bias:
        for name, n in (("bq", D.dq), ("bk", D.dkv), ("bv", D.dkv)):
            yield name, normal(seed, (l, name), (n,), 0.5, 0.0, torch.float32)


def ends_weights(D, seed, vocab):
    return (normal(seed, "embedding", (vocab, D.d)), normal(seed, "final_norm", (D.d,), 0.02, 1.0, torch.float32),
            normal(seed, "lm_head", (D.d, vocab), 0.02))


def packed_cache(D, seed, l, which, tokens):
    return normal(seed, (l, which), (tokens, D.hkv, D.dh))


def deal_pages(seed, lens, width):
    """Block tables: a random permutation of the pages (an eighth of them spare) dealt to the requests."""
    need = (lens + PAGE - 1) // PAGE
    pages = int(need.sum()) + max(1, int(need.sum()) // 8)
    perm = np.random.RandomState(number(seed, "pages") & 0x7FFFFFFF).permutation(pages)
    table = np.full((len(lens), width), -1, dtype=np.int32)
    at = 0
    for i, n in enumerate(need):
        table[i, :n] = perm[at:at + n]
        at += int(n)
    return table, pages


def on_gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def prefix(lens):
    return np.concatenate([[0], np.cumsum(lens)])


class Stage:
    """A stage of the library, given back when nothing refers to it or to its pools any more."""

    def __init__(self, config):
        self.handle = tdp.tdp_stage_create(config)

    def __del__(self):
        if getattr(self, "handle", None) is not None:
            tdp.tdp_stage_destroy(self.handle)


class Ends:
    def __init__(self, config):
        self.handle = tdp.tdp_ends_create(config)

    def __del__(self):
        if getattr(self, "handle", None) is not None:
            tdp.tdp_ends_destroy(self.handle)


class Raw:
    """Device memory of the library as an array.  A tensor made of it keeps it, and with it the memory's owner, alive."""

    def __init__(self, owner, address, count, kind):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": kind, "data": (address, False), "version": 2}


class State:
    """What an engine holds before the call."""


def make_stage(S, case, D, seed, pages, width, batch, tokens, seqs, weights=True):
    kv8 = case["kv8"]
    S.owner = Stage(tdp.StageConfig(
        n_layers=D.layers, d_model=D.d, n_q_heads=D.hq, n_kv_heads=D.hkv, head_dim=D.dh, d_ff=D.ff, rms_eps=D.eps,
        rope_base=D.base, page_size=PAGE, num_pages=pages, max_batch=batch, max_tokens=tokens, max_seqs=seqs,
        max_pages_per_seq=width, kv_dtype=tdp.KV_FP8_E4M3 if kv8 else tdp.KV_BF16, k_scale=K_SCALE if kv8 else 0.0,
        v_scale=V_SCALE if kv8 else 0.0, decode_micro_batches=0))
    S.stage = S.owner.handle
    for l in range(D.layers if weights else 0):
        for name, w in layer_weights(D, seed, l):
            tdp.tdp_stage_set_weight(S.stage, l, tdp.WEIGHT_IDS[name], w, tdp.BF16 if w.dtype == torch.bfloat16 else tdp.F32,
                                     tdp.DEVICE, w.shape[0], w.shape[1] if w.dim() == 2 else 1)
    S.pools = []
    for l in range(D.layers):
        k, v, n = tdp.tdp_stage_kv_pool(S.stage, l)
        for address in (k, v):
            if kv8:
                S.pools.append(torch.as_tensor(Raw(S.owner, address, n, "|u1"), device="cuda"))
            else:
                S.pools.append(torch.as_tensor(Raw(S.owner, address, n // 2, "<i2"), device="cuda").view(torch.bfloat16))


def make_ends(S, D, seed, vocab, rows):
    S.ends_owner = Ends(tdp.EndsConfig(vocab_size=vocab, d_model=D.d, rms_eps=D.eps, max_tokens=rows))
    S.ends = S.ends_owner.handle
    table, gain, head = ends_weights(D, seed, vocab)
    tdp.tdp_ends_set_weight(S.ends, tdp.E_EMBEDDING, table, tdp.BF16, tdp.DEVICE, vocab, D.d)
    tdp.tdp_ends_set_weight(S.ends, tdp.E_FINAL_NORM, gain, tdp.F32, tdp.DEVICE, D.d, 1)
    tdp.tdp_ends_set_weight(S.ends, tdp.E_LM_HEAD, head, tdp.BF16, tdp.DEVICE, D.d, vocab)
    S.logits = torch.empty((rows, vocab), dtype=torch.float32, device="cuda")
    S.tokens = torch.empty(rows, dtype=torch.int32, device="cuda")


def prepare(case, seed):
    S, D, kind = State(), Dims(case), case["kind"]
    S.kind, S.n = kind, case["n"]
    if kind == "head":
        make_ends(S, D, seed, case["vocab"], S.n)
        S.x = normal(seed, "hidden", (S.n, D.d))
        torch.cuda.synchronize()
        return S
    lens = lengths(case)
    most = D.prompt[2] if kind == "prefill" else D.ctx[2]
    width = (most + PAGE) // PAGE  # the longest request and its next token
    if kind == "prefill":
        S.total = int(lens.sum())
        table, pages = deal_pages(seed, lens, width)
        make_stage(S, case, D, seed, pages, width, 0, S.total, S.n)
        S.cu = on_gpu(prefix(lens))
        S.x = normal(seed, "hidden", (S.total, D.d))
    elif kind == "move":
        n = S.n
        table, pages = deal_pages(seed, lens, width)
        make_stage(S, case, D, seed, pages, width, 1, 0, 0, weights=False)
        S.t_in, S.t_out = int(lens[:n].sum()), int(lens[n:].sum())
        S.cu_in, S.cu_out = on_gpu(prefix(lens[:n])), on_gpu(prefix(lens[n:]))
        S.k_in, S.v_in = packed_cache(D, seed, "in", "k", S.t_in), packed_cache(D, seed, "in", "v", S.t_in)
        S.k_out, S.v_out = packed_cache(D, seed, "out", "k", S.t_out), packed_cache(D, seed, "out", "v", S.t_out)
        S.tab_in, S.tab_out = on_gpu(table[:n]), on_gpu(table[n:])
        tdp.tdp_stage_kv_import(S.stage, 0, S.k_out, S.v_out, S.cu_out, S.tab_out, n, S.t_out)
        torch.cuda.synchronize()
        S.k_out, S.v_out = torch.empty_like(S.k_out), torch.empty_like(S.v_out)
        torch.cuda.synchronize()
        return S
    else:  # decode, step: a cache as earlier calls left it
        table, pages = deal_pages(seed, lens + 1, width)
        make_stage(S, case, D, seed, pages, width, S.n, 0, 0)
        S.ctx = on_gpu(lens)
        cu, total = on_gpu(prefix(lens)), int(lens.sum())
        tab = on_gpu(table)
        for l in range(D.layers):
            tdp.tdp_stage_kv_import(S.stage, l, packed_cache(D, seed, l, "k", total), packed_cache(D, seed, l, "v", total),
                                    cu, tab, S.n, total)
        if kind == "step":
            make_ends(S, D, seed, case["vocab"], S.n)
            S.ids = on_gpu(np.random.RandomState(number(seed, "ids") & 0x7FFFFFFF).randint(0, case["vocab"], S.n))
            S.x = torch.empty((S.n, D.d), dtype=torch.bfloat16, device="cuda")
        else:
            S.x = normal(seed, "hidden", (S.n, D.d))
    S.table = on_gpu(table)
    S.y = torch.empty_like(S.x)
    torch.cuda.synchronize()
    return S


def run(S):
    if S.kind == "head":
        tdp.tdp_lm_head(S.ends, S.x, S.n, None, S.n, S.logits, S.tokens)
        return {"logits": S.logits, "tokens": S.tokens}
    if S.kind == "move":
        tdp.tdp_stage_kv_import(S.stage, 0, S.k_in, S.v_in, S.cu_in, S.tab_in, S.n, S.t_in)
        tdp.tdp_stage_kv_export(S.stage, 0, S.k_out, S.v_out, S.cu_out, S.tab_out, S.n, S.t_out)
        return {"k": S.k_out, "v": S.v_out, "pools": S.pools}
    if S.kind == "prefill":
        tdp.tdp_stage_prefill(S.stage, S.x, S.cu, S.table, S.n, S.total, S.y)
        return {"hidden": S.y, "pools": S.pools}
    if S.kind == "step":
        tdp.tdp_embed_tokens(S.ends, S.ids, S.n, S.x)
        tdp.tdp_stage_decode(S.stage, S.x, S.ctx, S.table, S.n, S.y)
        tdp.tdp_lm_head(S.ends, S.y, S.n, None, S.n, S.logits, S.tokens)
        return {"logits": S.logits, "tokens": S.tokens, "hidden": S.y, "pools": S.pools}
    tdp.tdp_stage_decode(S.stage, S.x, S.ctx, S.table, S.n, S.y)
    return {"hidden": S.y, "pools": S.pools}


def work(case):
    D, kind, n = Dims(case), case["kind"], case["n"]
    head = {"bytes": 0, "flops": 0}
    if kind in ("head", "step"):
        head = {"bytes": 2 * D.d * case["vocab"] + 4 * D.d + n * (2 * D.d + 4 * case["vocab"] + 4), "flops": 2 * n * D.d * case["vocab"]}
        if kind == "head":
            return head
    lens = lengths(case)
    cached = 2 * D.dkv * (1 if case["kv8"] else 2)  # one token's keys and values, one layer
    if kind == "move":
        return {"bytes": int(lens.sum()) * (cached + 4 * D.dkv), "flops": 0}
    weights = D.layers * (2 * D.params + 8 * D.d)
    if kind == "prefill":
        total = int(lens.sum())
        return {"bytes": weights + D.layers * cached * total + 4 * D.d * total,
                "flops": D.layers * (2 * total * D.params + sum(2 * D.dq * int(L) * (int(L) + 1) for L in lens))}
    span = int(lens.sum()) + n
    return {"bytes": weights + D.layers * cached * (span + n) + 4 * D.d * n + head["bytes"],
            "flops": D.layers * (2 * n * D.params + 4 * D.dq * span) + head["flops"]}


# bf16 operands, fp32 accumulation: about four times the distance measured between the kernels and the 64-bit result
# (decode 4e-3 to 5.5e-3, prefill 5e-3 to 9.3e-3, logits behind four layers 6e-3, the head alone 1.7e-3, toy widths
# 1.7e-3).  With an 8-bit cache values beside the middle of two codes add to it (decode 9e-3, prefill 1.8e-2).
REL = {"decode": 2e-2, "prefill": 3e-2, "head": 7e-3, "step": 2.4e-2}


def tolerance(case):
    kind = case["kind"]
    if kind == "move":
        return "exact"  # copies, and codes that are whole numbers
    t = {"rel": REL[kind]}
    if kind != "head" and case["kv8"]:
        t["rel"] = 3e-2
    elif case["shape"].startswith("tiny"):
        t["rel"] = 1e-2 if kind == "step" else 7e-3
    if kind in ("head", "step"):
        t["differ"] = 0.01  # the two largest logits of a row can lie closer than rounding
    elif case["kv8"]:
        t["differ"] = 0.005  # a value beside the middle of two codes can take either
    return t


# ---- the same in 64 bits, in plain torch ------------------------------------------------------------------------

def norm64(x, g, eps):
    return x * g / torch.sqrt((x * x).mean(-1, keepdim=True) + eps)


def rope64(z, pos, base):
    half = z.shape[-1] // 2
    theta = base ** (-torch.arange(half, dtype=torch.float64, device=z.device) * 2.0 / z.shape[-1])
    ang = pos.to(torch.float64)[:, None, None] * theta
    a, b = z[..., :half], z[..., half:]
    return torch.cat([a * ang.cos() - b * ang.sin(), a * ang.sin() + b * ang.cos()], dim=-1)


def codes64(x, scale):
    """What an 8-bit cache returns for x."""
    q = (x.float() / scale).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return q.to(torch.float64) * scale


def exact(case, seed):
    D, kind, n = Dims(case), case["kind"], case["n"]
    wide = torch.float64
    if kind == "move":
        lens = lengths(case)
        k = packed_cache(D, seed, "out", "k", int(lens[n:].sum()))
        v = packed_cache(D, seed, "out", "v", int(lens[n:].sum()))
        if case["kv8"]:
            k, v = codes64(k, K_SCALE).to(torch.bfloat16), codes64(v, V_SCALE).to(torch.bfloat16)
        return {"k": k.to(wide), "v": v.to(wide), "pools": [None, None]}
    if kind == "step":
        ids = torch.from_numpy(np.random.RandomState(number(seed, "ids") & 0x7FFFFFFF).randint(0, case["vocab"], n)).cuda()
        x = ends_weights(D, seed, case["vocab"])[0][ids].to(wide)
    elif kind != "head":
        lens = lengths(case)
        x = normal(seed, "hidden", (int(lens.sum()) if kind == "prefill" else n, D.d)).to(wide)
    else:
        x = normal(seed, "hidden", (n, D.d)).to(wide)
    if kind != "head":
        lens = lengths(case)
        cu = prefix(lens)
        if kind == "prefill":
            pos = torch.cat([torch.arange(int(L)) for L in lens]).cuda()
        else:
            pos = torch.from_numpy(lens).cuda()
        G = D.hq // D.hkv
        for l in range(D.layers):
            w = {name: t.to(wide) for name, t in layer_weights(D, seed, l)}
            y = norm64(x, w["g_attn"], D.eps)
            q, k, v = (y @ w[m] + w.get(b, 0.0) for m, b in (("wq", "bq"), ("wk", "bk"), ("wv", "bv")))
            q = rope64(q.view(-1, D.hq, D.dh), pos, D.base)
            k = rope64(k.view(-1, D.hkv, D.dh), pos, D.base)
            v = v.view(-1, D.hkv, D.dh)
            if case["kv8"]:
                k, v = codes64(k, K_SCALE), codes64(v, V_SCALE)
            a = torch.empty_like(q)
            if kind != "prefill":
                kc, vc = packed_cache(D, seed, l, "k", int(lens.sum())), packed_cache(D, seed, l, "v", int(lens.sum()))
            for i in range(n):
                lo, hi = int(cu[i]), int(cu[i + 1])
                if kind == "prefill":
                    seen = torch.ones(hi - lo, hi - lo, dtype=torch.bool, device="cuda").tril()
                    for h in range(D.hkv):
                        qi = q[lo:hi, h * G:(h + 1) * G].transpose(0, 1)
                        s = torch.matmul(qi, k[lo:hi, h].t().contiguous()) / math.sqrt(D.dh)
                        p = s.masked_fill_(~seen, -math.inf).softmax(-1)
                        a[lo:hi, h * G:(h + 1) * G] = torch.matmul(p, v[lo:hi, h].contiguous()).transpose(0, 1)
                        del s, p
                else:
                    ki, vi = kc[lo:hi].to(wide), vc[lo:hi].to(wide)
                    if case["kv8"]:
                        ki, vi = codes64(ki, K_SCALE), codes64(vi, V_SCALE)
                    ki, vi = torch.cat([ki, k[i:i + 1]]), torch.cat([vi, v[i:i + 1]])
                    qi = q[i].view(D.hkv, G, D.dh)
                    p = (torch.matmul(qi, ki.permute(1, 2, 0).contiguous()) / math.sqrt(D.dh)).softmax(-1)
                    a[i] = torch.matmul(p, vi.transpose(0, 1).contiguous()).reshape(D.hq, D.dh)
            x = x + a.reshape(-1, D.dq) @ w["wo"]
            y = norm64(x, w["g_mlp"], D.eps)
            x = x + (torch.nn.functional.silu(y @ w["wg"]) * (y @ w["wu"])) @ w["wd"]
            del w, y, q, k, v, a
        pools = [None] * (2 * D.layers)
        if kind != "step":
            return {"hidden": x, "pools": pools}
    _, gain, head = ends_weights(D, seed, case["vocab"])
    logits = norm64(x, gain.to(wide), D.eps) @ head.to(wide)
    if kind == "head":
        return {"logits": logits, "tokens": None}
    return {"logits": logits, "tokens": None, "hidden": x, "pools": pools}
