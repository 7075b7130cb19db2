"""The measured cases of the Jacobi-step engine.

Every case goes through the C ABI of include/jf.h as a user's program calls
it: a model's step, multi-block step, packed forward or prefill, and the
attention, LM-head and trajectory calls.  Most cases run a few decoder layers
of a model's dimensions with a small vocabulary (the layers are what a step
repeats); two run the whole 28-layer shape with its full vocabulary.

Inputs are made on the GPU from the seed alone.  The draft rows are drawn
tokens, the first one too (a caller that forces the continuation), so that no
input depends on an argmax.  Model cases return the step's logits and the KV
cache the step wrote, not the tokens: a near-tie between two logits may swap
one of a few rows' tokens under any change of rounding.
"""
import ctypes
import math

import torch

from paper_2512_14681_amd import jf

# Decoder dimensions (d_model, query heads, KV heads, head_dim, d_ffn, RoPE base).
DIMS = {
    "7b": (3584, 28, 4, 128, 18944, 1e6),    # the benchmark's decoder shape
    "mid": (2048, 16, 4, 128, 8192, 1e6),    # the mid-size bf16 decoder of the tests
    "small": (1024, 16, 2, 64, 2816, 1e4),   # generic: head_dim 64, an FFN that is no power of two
    "tiny": (128, 4, 4, 32, 512, 1e4),       # the tests' fp32 decoder
}
EPS = 1e-6
PAGE = 64


def listed():
    return [
        # One step of a tiny fp32 decoder in block mode: the smallest call, launches and host time.
        {"name": "step_tiny_f32_rows8", "kind": "step", "dims": "tiny", "dtype": "f32", "layers": 2, "vocab": 1024,
         "prefix": 32, "rows": 8, "mode": 0, "max_rows": 16},
        # One row: greedy decoding, and the last step of a block.
        {"name": "step_rows1", "kind": "step", "dims": "7b", "dtype": "bf16", "layers": 2, "vocab": 8192,
         "prefix": 1024, "rows": 1, "mode": 0, "max_rows": 64},
        # Block mode partly accepted: an odd number of rows at an odd length, a smaller decoder.
        {"name": "step_mid_rows13", "kind": "step", "dims": "mid", "dtype": "bf16", "layers": 2, "vocab": 8192,
         "prefix": 777, "rows": 13, "mode": 0, "max_rows": 64},
        # A running window of 64 tokens.
        {"name": "step_rows64", "kind": "step", "dims": "7b", "dtype": "bf16", "layers": 2, "vocab": 8192,
         "prefix": 1024, "rows": 64, "mode": 1, "max_rows": 64},
        # The paper's configuration: block 64, 2 blocks, verification size 4: 320 rows under the tree mask.
        {"name": "multiblock_rows320", "kind": "multiblock", "dims": "7b", "dtype": "bf16", "layers": 2,
         "vocab": 8192, "prefix": 1024, "n": 64, "blocks": 2, "cands": 3, "max_rows": 320},
        # A packed training sequence of 8 noisy and 8 clean blocks of 16.
        {"name": "packed_rows256", "kind": "packed", "dims": "7b", "dtype": "bf16", "layers": 2, "vocab": 8192,
         "prefix": 1024, "n": 16, "blocks": 8, "mask": 0, "max_rows": 256},
        # A ragged prompt of 1000 tokens into an empty cache.
        {"name": "prefill_1000", "kind": "prefill", "dims": "7b", "dtype": "bf16", "layers": 2, "vocab": 8192,
         "prefix": 1000, "max_rows": 512},
        # The attention of one layer over a long, ragged prefix under a tree mask.
        {"name": "attention_8000x48", "kind": "attention", "dims": "7b", "dtype": "bf16", "prefix": 8000, "rows": 48,
         "tree": True},
        # The LM head with acceptance at the full vocabulary.
        {"name": "lm_head_rows64", "kind": "lm_head", "d": 3584, "vocab": 152064, "dtype": "bf16", "rows": 64},
        # Noise-schedule point selection over the trajectories of a collection run.
        {"name": "trajectory_select_16", "kind": "select", "blocks": 1 << 18, "n": 16, "w": 16, "counts": False},
        # The whole decoder: the headline step, a 16-token window after 1024 tokens.
        {"name": "step_7b_rows16", "kind": "step", "dims": "7b", "dtype": "bf16", "layers": 28, "vocab": 152064,
         "prefix": 1024, "rows": 16, "mode": 1, "max_rows": 64},
        # The whole decoder: a full multi-block step, 4 blocks of 16 and 8 recycled candidates after 2048 tokens.
        {"name": "multiblock_7b_rows192", "kind": "multiblock", "dims": "7b", "dtype": "bf16", "layers": 28,
         "vocab": 152064, "prefix": 2048, "n": 16, "blocks": 4, "cands": 8, "max_rows": 192},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(["step", "multiblock", "packed", "prefill", "attention", "lm_head", "select"],
                       [8, 3, 2, 3, 3, 3, 2])[0]
    if kind == "select":
        return {"kind": kind, "blocks": _log_int(rng, 1 << 10, 1 << 18), "n": rng.choice([8, 16, 16, 24, 32]),
                "w": rng.choice([8, 16, 16, 31]), "counts": rng.random() < 0.3}
    if kind == "lm_head":
        return {"kind": kind, "d": rng.choice([1024, 2048, 3584]), "vocab": 16 * _log_int(rng, 512, 9504),
                "dtype": "bf16", "rows": _log_int(rng, 1, 512)}
    if kind == "attention":
        dims = rng.choice(["7b", "7b", "mid", "small"])
        return {"kind": kind, "dims": dims, "dtype": "f32" if rng.random() < 0.15 else "bf16",
                "prefix": _log_int(rng, 100, 8192), "rows": _log_int(rng, 1, 320), "tree": rng.random() < 0.5}
    dims = rng.choice(["7b", "7b", "7b", "mid", "mid", "small", "tiny"])
    c = {"kind": kind, "dims": dims, "dtype": "f32" if dims == "tiny" else "bf16", "layers": rng.randint(1, 3),
         "vocab": rng.choice([1024, 8192, 32000]), "prefix": _log_int(rng, 20, 2500)}
    if kind == "step":
        c["rows"] = _log_int(rng, 1, 512)
        c["mode"] = rng.randint(0, 1)
        c["max_rows"] = max(64, c["rows"])
    elif kind == "multiblock":
        c["n"] = rng.choice([8, 16, 16, 21, 32, 64])
        c["blocks"] = rng.randint(1, 4)
        c["cands"] = rng.randint(0, 8)
        while c["n"] * (c["blocks"] + c["cands"]) > 512:
            c["blocks"], c["cands"] = max(1, c["blocks"] - 1), max(0, c["cands"] - 1)
        c["max_rows"] = c["n"] * (c["blocks"] + c["cands"])
    elif kind == "packed":
        c["n"] = rng.choice([5, 8, 16, 16, 32])
        c["blocks"] = _log_int(rng, 1, 256 // c["n"])
        c["mask"] = rng.randint(0, 1)
        c["max_rows"] = max(64, 2 * c["n"] * c["blocks"])
    else:
        c["max_rows"] = rng.choice([64, 192, 256, 512])
    return c


# ---- shapes ---------------------------------------------------------------------------
def _shape(case):
    d, H, G, hd, F, base = DIMS[case["dims"]]
    return {"d_model": d, "n_heads": H, "n_kv_heads": G, "head_dim": hd, "d_ffn": F, "rope_base": base,
            "rms_eps": EPS, "n_layers": case.get("layers", 1), "vocab": case.get("vocab", 16), "dtype": case["dtype"]}


def _rows(case):
    """In-step rows of a model case (a prefill has none)."""
    k = case["kind"]
    if k == "step":
        return case["rows"]
    if k == "multiblock":
        return case["n"] * (case["blocks"] + case["cands"])
    return 2 * case["n"] * case["blocks"] if k == "packed" else 0


def _segments(case):
    """The draft, its pseudo-active blocks in a chain behind it, the recycled candidates under the draft's first row."""
    n, K = case["n"], case["blocks"]
    segs = [(0, n, -1, jf.JF_ROLE_RA, 1)]
    segs += [(b * n, n, b * n - 1, jf.JF_ROLE_PSEUDO, 0) for b in range(1, K)]
    return segs + [((K + c) * n, n, 0, jf.JF_ROLE_CAND, 0) for c in range(case["cands"])]


def _parents(case):
    """The parent row of every in-step row (-1: a root)."""
    k, R = case["kind"], _rows(case) if "rows" not in case else case["rows"]
    if k == "multiblock":
        par = []
        for first, n, attach, _, _ in _segments(case):
            par += [attach] + list(range(first, first + n - 1))
        return par
    if k == "packed":
        n, par = case["n"], []
        for b in range(case["blocks"]):
            for copy in (0, 1):
                clean = copy == 1 or case["mask"] == jf.JF_MASK_CLEAN_CONTEXT
                root = -1 if b == 0 else (2 * b * n - 1 if clean else (2 * b - 1) * n - 1)
                par += [root] + [(2 * b + copy) * n + i for i in range(n - 1)]
        return par
    if k == "attention" and case["tree"]:  # half the rows a chain, the rest branches of 8 under its first row
        return [r - 1 if r < (R + 1) // 2 or (r - (R + 1) // 2) % 8 else 0 for r in range(R)]
    return list(range(-1, R - 1))


def _forest(case):
    """(visibility [R][R] bool: ancestors and the row itself, depth [R]) on the CPU."""
    par = _parents(case)
    R = len(par)
    vis, depth = torch.zeros(R, R, dtype=torch.bool), torch.zeros(R, dtype=torch.int64)
    for r, p in enumerate(par):
        if p >= 0:
            vis[r] = vis[p]
            depth[r] = depth[p] + 1
        vis[r, r] = True
    return vis, depth


# ---- inputs ---------------------------------------------------------------------------
def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + stream) & 0x7FFFFFFFFFFF)
    return g


def _dt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _normal(g, *shape, std=1.0, mean=0.0, dtype=torch.float32):
    return torch.empty(*shape, dtype=dtype, device="cuda").normal_(mean, std, generator=g)


def _weights(case, seed):
    """The model's tensors in the order jf_model_load takes them: N(0, 0.02), norm gains 1 + 0.1 N(0, 1)."""
    s, g, dt = _shape(case), _gen(seed, 1), _dt(case)
    d, H, G, hd, F, V = (s[k] for k in ("d_model", "n_heads", "n_kv_heads", "head_dim", "d_ffn", "vocab"))
    w = lambda *shape: _normal(g, *shape, std=0.02, dtype=dt)  # noqa: E731
    gain = lambda: _normal(g, d, std=0.1, mean=1.0, dtype=dt)  # noqa: E731
    out = [w(V, d)]
    for _ in range(s["n_layers"]):
        out += [gain(), w(H * hd, d), w(G * hd, d), w(G * hd, d), w(d, H * hd), gain(), w(F, d), w(F, d), w(d, F)]
    return out + [gain(), w(V, d)]


def _tokens(case, seed):
    """(prompt, in-step rows) of a model case."""
    g = _gen(seed, 2)
    return (torch.randint(0, case["vocab"], (case["prefix"],), device="cuda", generator=g, dtype=torch.int32),
            torch.randint(0, case["vocab"], (_rows(case),), device="cuda", generator=g, dtype=torch.int32))


def _planes(x, case):
    """An fp32 tensor as activation planes: hi and lo bf16, or one fp32 plane."""
    if case["dtype"] == "f32":
        return x[None]
    hi = x.to(torch.bfloat16)
    return torch.stack([hi, (x - hi.float()).to(torch.bfloat16)])


def _gemm_layout(x):
    """[..., R, K] as the GEMM-input layout of include/jf.h: rows padded to 16 with zeros, 16 x 128 blocks in matrix-core order."""
    R, K = x.shape[-2:]
    Rp = (R + 15) // 16 * 16
    x = torch.nn.functional.pad(x, (0, 0, 0, Rp - R))
    x = x.reshape(*x.shape[:-2], Rp // 16, 16, K // 128, 4, 4, 8)
    n = x.dim() - 6
    return x.permute(*range(n), n, n + 2, n + 4, n + 3, n + 1, n + 5).reshape(*x.shape[:n], Rp * K).contiguous()


def _attention_inputs(case, seed):
    """q [R][H][hd] fp32 (as its planes hold it), keys and values [C + R][G][hd] of the cache's type, the page table."""
    d, H, G, hd, _, _ = DIMS[case["dims"]]
    g, T = _gen(seed, 3), case["prefix"] + case["rows"]
    q = _planes(_normal(g, case["rows"], H, hd), case)
    k, v = _normal(g, T, G, hd, dtype=_dt(case)), _normal(g, T, G, hd, dtype=_dt(case))
    return q, k, v, torch.randperm((T + PAGE - 1) // PAGE, device="cuda", generator=g).to(torch.int32)


def _pages(k, v, n_pages):
    """[T][G][hd] keys and values as n_pages logical pages: K [G][64][hd], then V transposed [G][hd][64]; zero past T."""
    T, G, hd = k.shape
    pad = lambda x: torch.nn.functional.pad(x, (0, 0, 0, 0, 0, n_pages * PAGE - T)).reshape(n_pages, PAGE, G, hd)  # noqa: E731
    return torch.cat([pad(k).permute(0, 2, 1, 3).reshape(n_pages, -1), pad(v).permute(0, 2, 3, 1).reshape(n_pages, -1)], 1)


class _Model:
    """The caller's buffers of one loaded model."""

    def __init__(self, case, seed):
        C, R = case["prefix"], _rows(case)
        max_rows = max(case["max_rows"], R)
        self.cfg = jf.config(_shape(case), max_rows, (C + R + PAGE - 1) // PAGE * PAGE)
        sizes = jf.query_sizes(self.cfg)
        self.packed, self.kv_bytes, self.ws = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in sizes)
        w = _weights(case, seed)
        ptrs = (ctypes.c_void_p * len(w))(*[t.data_ptr() for t in w])
        h = ctypes.c_void_p()
        jf.check(jf.lib().jf_model_load(ctypes.byref(self.cfg), ptrs, len(w), jf._ptr(self.packed),
                                        jf._ptr(self.kv_bytes), jf._ptr(self.ws), jf._stream(), ctypes.byref(h)))
        self.h = h
        self.kv = self.kv_bytes.view(_dt(case))

    def __del__(self):
        if getattr(self, "h", None):
            jf.lib().jf_model_free(self.h)
            self.h = None


def _ints(n):
    return torch.zeros(max(1, n), dtype=torch.int32, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "kind": kind}
    if kind == "select":
        g, B, n = _gen(seed, 4), case["blocks"], case["n"]
        # block b converges in k_b iterations: point j keeps a growing prefix of the fixed point, differs from it at
        # the next position, and beyond has its token with probability 1/4; the last two points are the fixed point
        k = torch.randint(1, n + 1, (B, 1, 1), device="cuda", generator=g, dtype=torch.int32)
        j = torch.arange(n + 1, device="cuda", dtype=torch.int32).view(1, -1, 1)
        p = torch.arange(n, device="cuda", dtype=torch.int32).view(1, 1, -1)
        m = 1 + (j * (n - 1)) // (k - 1).clamp(min=1)
        fixed = torch.randint(0, 152064, (B, 1, n), device="cuda", generator=g, dtype=torch.int32)
        other = torch.randint(0, 152064, (B, n + 1, n), device="cuda", generator=g, dtype=torch.int32)
        t = torch.where(other % 4 == 0, fixed, other)
        t = torch.where(p == m, (fixed + 1 + other % 152063) % 152064, t)
        t = torch.where((p < m) | (j >= k - 1), fixed, t)
        s["traj"] = torch.where(j > k, -1, t).to(torch.int32).contiguous()
        s["len"] = (k + 1).reshape(B).contiguous()
        s["sel"] = _ints(B)
        s["unconv"] = torch.zeros(B, n + 1, dtype=torch.int32, device="cuda") if case["counts"] else None
        return s
    if kind == "lm_head":
        g, R, d, V, dt = _gen(seed, 5), case["rows"], case["d"], case["vocab"], _dt(case)
        code = jf.JF_BF16 if case["dtype"] == "bf16" else jf.JF_F32
        w = _normal(g, V, d, std=0.02, dtype=dt)
        L, st = jf.lib(), jf._stream()
        s["w"] = torch.empty(L.jf_packed_matrix_bytes(V, d, code), dtype=torch.uint8, device="cuda")
        jf.check(L.jf_pack_matrix(V, d, code, jf._ptr(w), jf._ptr(s["w"]), st))
        s["x"] = _gemm_layout(_planes(_normal(g, R, d), case))
        s["argmax"], s["result"], s["logits"] = _ints(R), _ints(4), torch.zeros(R, V, device="cuda")
        s["ws"] = torch.empty(L.jf_lm_head_ws_bytes(R, V), dtype=torch.uint8, device="cuda")
        # a draft that is accepted up to its middle
        jf.check(L.jf_lm_head_accept(R, d, V, code, jf._ptr(s["x"]), jf._ptr(s["w"]), None, jf._ptr(s["argmax"]), None,
                                     None, jf._ptr(s["ws"]), st))
        s["draft"] = torch.cat([s["argmax"][:1], s["argmax"][:-1]]).contiguous()
        s["draft"][R // 2] = (s["draft"][R // 2] + 1) % V
        s["code"] = code
        return s
    if kind == "attention":
        _, H, G, hd, _, _ = DIMS[case["dims"]]
        R = case["rows"]
        q, k, v, pt = _attention_inputs(case, seed)
        pages = _pages(k, v, len(pt))
        s["kv"] = torch.empty_like(pages)
        s["kv"][pt.long()] = pages          # logical page p at physical page pt[p]
        s["q"], s["pt"] = q.contiguous(), pt
        s["vis"] = None
        if case["tree"]:
            bits = torch.zeros(R, 64 * jf.JF_VIS_WORDS, dtype=torch.bool)
            bits[:, :R] = _forest(case)[0]
            weights = (torch.ones(64, dtype=torch.int64) << torch.arange(64)).view(1, 1, 64)
            s["vis"] = (bits.view(R, jf.JF_VIS_WORDS, 64).long() * weights).sum(2).contiguous().cuda()
        s["out"] = torch.zeros(q.shape[0], (R + 15) // 16 * 16 * H * hd, dtype=_dt(case), device="cuda")
        s["ws"] = torch.empty(jf.lib().jf_attention_ws_bytes(H, hd, R), dtype=torch.uint8, device="cuda")
        s["code"] = jf.JF_BF16 if case["dtype"] == "bf16" else jf.JF_F32
        return s
    s["m"] = m = _Model(case, seed)
    R = _rows(case)
    s["prompt"], s["tokens"] = _tokens(case, seed)
    s["pending"] = _ints(1)
    jf.check(jf.lib().jf_prefill(m.h, jf._ptr(s["prompt"]), case["prefix"], jf._ptr(s["pending"]), jf._stream()))
    if R:
        s["argmax"], s["result"], s["next"], s["path"] = _ints(R), _ints(4), _ints(R), _ints(R)
        s["accept"] = _ints(jf.JF_MAX_SEGMENTS)
        s["logits"] = torch.zeros(R, case["vocab"], device="cuda")
    if kind == "multiblock":
        s["segs"] = jf.segments(_segments(case))
    return s


def run(s):
    c, kind, L, st, p = s["case"], s["kind"], jf.lib(), jf._stream(), jf._ptr
    if kind == "select":
        jf.trajectory_select(s["traj"], s["len"], c["blocks"], c["n"], c["n"] + 1, c["w"], s["sel"], d_unconv=s["unconv"])
        return [s["sel"], s["unconv"]]
    if kind == "lm_head":
        jf.check(L.jf_lm_head_accept(c["rows"], c["d"], c["vocab"], s["code"], p(s["x"]), p(s["w"]), p(s["draft"]),
                                     p(s["argmax"]), p(s["result"]), p(s["logits"]), p(s["ws"]), st))
        return [s["logits"], s["argmax"], s["result"]]
    if kind == "attention":
        _, H, G, hd, _, _ = DIMS[c["dims"]]
        jf.check(L.jf_attention(H, G, hd, s["code"], c["prefix"], c["rows"], p(s["q"]), p(s["kv"]), p(s["pt"]),
                                p(s["vis"]), p(s["out"]), p(s["ws"]), st))
        # the value the planes stand for
        return [torch.sum(s["out"], 0, dtype=torch.float32)]
    m = s["m"]
    if kind == "prefill":
        jf.check(L.jf_kv_truncate(m.h, 0, st))
        jf.check(L.jf_prefill(m.h, p(s["prompt"]), c["prefix"], p(s["pending"]), st))
        return [m.kv]
    if kind == "step":
        jf.check(L.jf_jacobi_step(m.h, p(s["tokens"]), c["rows"], c["mode"], 2, p(s["argmax"]), p(s["result"]),
                                  p(s["next"]), p(s["logits"]), st))
    elif kind == "multiblock":
        jf.check(L.jf_multiblock_step(m.h, p(s["tokens"]), _rows(c), s["segs"], len(s["segs"]), p(s["argmax"]),
                                      p(s["accept"]), p(s["result"]), p(s["path"]), p(s["logits"]), st))
    else:
        jf.check(L.jf_packed_forward(m.h, p(s["tokens"]), c["blocks"], c["n"], c["mask"], p(s["argmax"]),
                                     p(s["logits"]), st))
    return [s["logits"], m.kv]


# ---- what a pass cannot do without ----------------------------------------------------
def work(case):
    kind, e = case["kind"], 2 if case.get("dtype") == "bf16" else 4
    if kind == "select":  # every valid point, the lengths, the selections; (n + 3) / 2 points a block on average
        B, n = case["blocks"], case["n"]
        b = B * ((n + 3) / 2 * n * 4 + 8) + (B * (n + 1) * 4 if case["counts"] else 0)
        return {"bytes": b, "flops": B * (n + 3) / 2 * n}
    if kind == "lm_head":
        R, d, V = case["rows"], case["d"], case["vocab"]
        return {"bytes": V * d * e + R * d * 4 + R * V * 4, "flops": 2 * R * V * d}
    d, H, G, hd, F, _ = DIMS[case["dims"]]
    C, R = case["prefix"], case["rows"] if kind == "attention" else _rows(case)
    if kind == "prefill":
        C, R = 0, C
    pairs = R * C + (R * (R + 1) // 2 if kind in ("step", "prefill") else int(_forest(case)[0].sum()))
    att = {"bytes": (C + R) * G * hd * 2 * e, "flops": 4 * H * hd * pairs}
    if kind == "attention":
        return {"bytes": att["bytes"] + R * H * hd * 8, "flops": att["flops"]}
    layer = (H + 2 * G) * hd * d + d * H * hd + 3 * F * d
    V, n = case["vocab"], case["layers"]
    head = 1 if kind == "prefill" else R          # a prefill reads the head for its last row
    by = n * (layer * e + att["bytes"]) + V * d * e + R * d * e + (0 if kind == "prefill" else R * V * 4)
    return {"bytes": by, "flops": n * (2 * layer * R + att["flops"]) + 2 * V * d * head}


def tolerance(case):
    """About four times the error measured against exact()."""
    kind = case["kind"]
    if kind == "select":
        return "exact"
    if case["dtype"] == "f32":  # fp32 sums: 2.5e-7 to 3.5e-7
        return {"rel": 2e-6, "max": 1e-4}
    if kind == "lm_head":       # fp32 sums of 16-bit products: 5e-7; tokens swap at exact ties only
        return {"rel": 2e-6, "max": 1e-4, "differ": 0.01}
    if kind == "attention":     # Q and P as two 16-bit terms: 3e-6
        return {"rel": 1.5e-5, "max": 1e-3}
    # K/V entries that round to the neighbouring bf16 value: 4e-4 after 2 or 3 layers, 1.2e-3 after 28
    return {"rel": 1.5e-3 if case["layers"] <= 3 else 5e-3, "max": 0.1}


# ---- the same in 64 bits --------------------------------------------------------------
def _attend(q, k, v, mask):
    """q [R][H][hd]; k, v [T][G][hd]; mask [R][T]: softmax(q k^T / sqrt(hd)) v, query head j on KV head j // (H / G)."""
    R, H, hd = q.shape
    G = k.shape[1]
    out = torch.empty_like(q)
    for r0 in range(0, R, 512):
        mk = mask[r0:r0 + 512]
        for h in range(H):
            kh, vh = k[:, h // (H // G)], v[:, h // (H // G)]
            sc = (q[r0:r0 + 512, h] @ kh.t().contiguous()) / math.sqrt(hd)
            out[r0:r0 + 512, h] = torch.softmax(sc.masked_fill(~mk, -math.inf), 1) @ vh.contiguous()
    return out


def _mm(x, w):
    """x W^T in 64 bits, the weight in slices."""
    return torch.cat([x @ w[i:i + 8192].double().t() for i in range(0, len(w), 8192)], 1)


def _norm(h, gain):
    return h / torch.sqrt((h * h).mean(1, keepdim=True) + EPS) * gain.double()


def exact(case, seed):
    kind, f64 = case["kind"], torch.float64
    if kind == "select":
        return None
    if kind == "lm_head":
        g, R, d, V = _gen(seed, 5), case["rows"], case["d"], case["vocab"]
        w = _normal(g, V, d, std=0.02, dtype=_dt(case))
        return [_mm(_planes(_normal(g, R, d), case).to(f64).sum(0), w), None, None]
    d, H, G, hd, F, base = DIMS[case["dims"]]
    C = case["prefix"]
    R = case["rows"] if kind == "attention" else _rows(case)
    T = C + R
    vis, depth = (t.cuda() for t in _forest(case)) if R else (None, None)
    if kind == "attention":
        q, k, v, _ = _attention_inputs(case, seed)
        mask = torch.cat([torch.ones(R, C, dtype=torch.bool, device="cuda"), vis], 1)
        o = _attend(q.to(f64).sum(0), k.to(f64), v.to(f64), mask)
        return [_gemm_layout(o.reshape(R, H * hd))]
    # the prompt's rows and the step's rows as one sequence: each sees what its call saw
    mask = torch.zeros(T, T, dtype=torch.bool, device="cuda")
    mask[:C, :C] = torch.tril(torch.ones(C, C, dtype=torch.bool, device="cuda"))
    pos = torch.arange(C, device="cuda")
    if R:
        mask[C:, :C] = True
        mask[C:, C:] = vis
        pos = torch.cat([pos, C + depth])
    w = _weights(case, seed)
    prompt, rows = _tokens(case, seed)
    h = w[0][torch.cat([prompt, rows]).long()].to(f64)
    half = hd // 2
    ang = pos[:, None].to(f64) * base ** (-2.0 * torch.arange(half, device="cuda", dtype=f64) / hd)
    cs, sn = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    rope = lambda x: torch.cat([x[..., :half] * cs - x[..., half:] * sn, x[..., half:] * cs + x[..., :half] * sn], -1)  # noqa: E731
    cached = lambda x: x.to(_dt(case)).to(f64)  # noqa: E731  (the cache holds the weights' type)
    n_pages = (T + PAGE - 1) // PAGE
    kv = []
    for l in range(case["layers"]):
        an, wq, wk, wv, wo, fn, wg, wu, wd = w[1 + 9 * l:10 + 9 * l]
        x = _norm(h, an)
        q = rope(_mm(x, wq).view(T, H, hd))
        k, v = cached(rope(_mm(x, wk).view(T, G, hd))), cached(_mm(x, wv).view(T, G, hd))
        kv.append(_pages(k, v, n_pages).reshape(-1))
        h = h + _mm(_attend(q, k, v, mask).view(T, H * hd), wo)
        x = _norm(h, fn)
        gate = _mm(x, wg)
        h = h + _mm(torch.nn.functional.silu(gate) * _mm(x, wu), wd)
    kv = torch.cat(kv)
    if kind == "prefill":
        return [kv]
    return [_mm(_norm(h[C:], w[-2]), w[-1]), kv]
