"""The calls that a decode-serving program makes of this framework, as cases that can be timed and checked.

Every case goes through the public binding (the C-ABI's entry points) or ``DecodeModel.step``:

* ``proj``   weight matrices of a layer, each one ``boost_decode_gemv`` call on its own activations;
* ``attn``   one layer's paged GQA decode attention over a filled KV pool;
* ``qkvo``   the attention half of a layer: embedding, norm, qkv, RoPE + KV append, attention, output
             projection, residual + norm;
* ``mlp``    the MLP half of a layer: embedding, norm, gate_up, SiLU, down, residual + norm;
* ``head``   the end of a step: embedding, norm, lm_head, argmax;
* ``step``   a whole decode step of a short model.

``modulus`` is the modulo placement's M (every M-th 2 MiB page on host; 130 is what calibration gives on this GPU,
16 the single-layer configuration's; 0 keeps everything in HBM).
"""
import math

import numpy as np
import torch

from paper_2609_13592_amd import binding as bd
from paper_2609_13592_amd.step import EPS, THETA, DecodeModel, Dims

HD = 128  # head dimension of every configuration here
EMBED_ROWS = 2048  # rows of the embedding table of the half-layer cases
QKVO_8B = "6144x4096,4096x4096,28672x4096,4096x14336"  # qkv, o, gate_up, down
QKVO_70B = "10240x8192,8192x8192,57344x8192,8192x28672"


def listed():
    return [
        # one linear layer with one of its 16 pages on host: the smallest tiered call, bound by the host link
        {"name": "single layer, host page", "kind": "proj", "shapes": "4096x4096", "batch": 1, "modulus": 16, "out": "f32"},
        # the matrices of an 8B layer at batch 1: the decode weight chain of bench.py, one layer of it
        {"name": "8B layer, batch 1", "kind": "proj", "shapes": QKVO_8B, "batch": 1, "modulus": 130, "out": "f32"},
        # the end of an 8B step at batch 1: the largest matrix, three of its pages on host, and the token choice
        {"name": "8B head, batch 1", "kind": "head", "d": 4096, "vocab": 128256, "batch": 1, "modulus": 130},
        # a small matrix of odd sizes, rows cut by page boundaries, a few requests, bf16 results
        {"name": "odd matrix, batch 5", "kind": "proj", "shapes": "5003x3080", "batch": 5, "modulus": 0, "out": "bf16"},
        # the matrices of a 70B layer at the batch of the capacity-capped configuration
        {"name": "70B layer, batch 8", "kind": "proj", "shapes": QKVO_70B, "batch": 8, "modulus": 130, "out": "f32"},
        # the MLP half of an 8B layer at the high-throughput configuration's batch
        {"name": "8B MLP, batch 64", "kind": "mlp", "d": 4096, "ffn": 14336, "batch": 64, "modulus": 130},
        # the matrices of an 8B layer at the largest batch
        {"name": "8B layer, batch 256", "kind": "proj", "shapes": QKVO_8B, "batch": 256, "modulus": 130, "out": "f32"},
        # the attention half of an 8B layer, a ragged batch with contexts from one token up
        {"name": "8B attention half, batch 33", "kind": "qkvo", "d": 4096, "q_heads": 32, "kv_heads": 8, "batch": 33,
         "ctx_lo": 1, "ctx_hi": 2500, "modulus": 130},
        # paged attention of the 64-request configuration
        {"name": "attention, batch 64", "kind": "attn", "q_heads": 32, "kv_heads": 8, "batch": 64,
         "ctx_lo": 512, "ctx_hi": 4096, "modulus": 130, "out": "f32"},
        # paged attention of the 70B-shaped configuration: eight query heads per KV head, few requests
        {"name": "70B attention, batch 8", "kind": "attn", "q_heads": 64, "kv_heads": 8, "batch": 8,
         "ctx_lo": 2048, "ctx_hi": 2048, "modulus": 130, "out": "bf16"},
        # one long request alone: the attention call with the fewest work items
        {"name": "attention, one request", "kind": "attn", "q_heads": 32, "kv_heads": 8, "batch": 1,
         "ctx_lo": 8192, "ctx_hi": 8192, "modulus": 130, "out": "bf16"},
        # a whole step: two layers of 8B dimensions and the head, a middling batch
        {"name": "8B step of 2 layers, batch 16", "kind": "step", "layers": 2, "d": 4096, "q_heads": 32, "kv_heads": 8,
         "ffn": 14336, "vocab": 32000, "batch": 16, "ctx_lo": 1024, "ctx_hi": 4096, "modulus": 130},
    ]


LARGEST = 1.7e9  # bytes of the largest listed case (the 70B layer)


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    kind = rng.choice(["proj"] * 7 + ["attn"] * 6 + ["qkvo"] * 2 + ["mlp"] * 2 + ["head"] * 2 + ["step"])
    # batches as they are served: few requests as often as many, round sizes and others
    batch = _log(rng, 1, 256)
    modulus = rng.choice([0, 130, 130])
    if kind == "proj":
        n, k = _log(rng, 300, 60000), 8 * _log(rng, 64, 3600)
        if rng.random() < 0.5:  # a model's sizes are multiples of 128
            n, k = max(128, n // 128 * 128), max(512, k // 128 * 128)
        if n * k <= 32 << 20 and rng.random() < 0.2:
            modulus = 16
        return {"kind": kind, "shapes": "%dx%d" % (n, k), "batch": batch, "modulus": modulus,
                "out": rng.choice(["f32", "f32", "bf16"])}
    group = rng.choice([1, 2, 4, 4, 8])
    kv_heads = rng.choice([2, 4, 8, 8])
    hi = _log(rng, 64, 8192)
    lo = rng.choice([1, max(1, hi // 8), hi])
    if kind == "attn":
        return {"kind": kind, "q_heads": group * kv_heads, "kv_heads": kv_heads, "batch": min(batch, 160),
                "ctx_lo": lo, "ctx_hi": hi, "modulus": modulus, "out": rng.choice(["f32", "bf16"])}
    d = rng.choice([1024, 2048, 4096, 4096, 5120, 8192])
    ffn = 128 * _log(rng, 16, 160)
    if kind == "qkvo":
        return {"kind": kind, "d": d, "q_heads": group * kv_heads, "kv_heads": kv_heads, "batch": min(batch, 100),
                "ctx_lo": lo, "ctx_hi": min(hi, 4096) if lo < hi else lo, "modulus": modulus}
    if kind == "mlp":
        return {"kind": kind, "d": d, "ffn": ffn, "batch": batch, "modulus": modulus}
    vocab = rng.choice([32000, 32003, 128256, 151936])
    if kind == "head":
        return {"kind": kind, "d": d, "vocab": vocab, "batch": min(batch, 64), "modulus": modulus}
    return {"kind": kind, "layers": rng.choice([1, 2]), "d": min(d, 4096), "q_heads": group * kv_heads,
            "kv_heads": kv_heads, "ffn": ffn, "vocab": 32000, "batch": min(batch, 48), "ctx_lo": min(lo, 2048),
            "ctx_hi": min(hi, 2048), "modulus": modulus}


def draw(rng):
    while True:
        c = _draw(rng)
        if c.get("ctx_lo", 0) <= c.get("ctx_hi", 0) and work(c)["bytes"] <= LARGEST and work(c)["flops"] <= 5e11:
            return c


# ---------------------------------------------------------------------------------------------- inputs
def _shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["shapes"].split(",")]


def _dims(case):
    return Dims(layers=case.get("layers", 1), d=case["d"], hq=case.get("q_heads", 1), hkv=case.get("kv_heads", 1),
                hd=HD, ffn=case.get("ffn", 8), vocab=case.get("vocab", EMBED_ROWS))


def _normal(seed, what, shape, sigma=1.0):
    """bf16 ~N(0, sigma) on the GPU, a stream of its own for every (seed, what)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1009 + what)
    t = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    return (t if sigma == 1.0 else t.mul_(sigma)).to(torch.bfloat16)


def _lens(case, seed):
    """Context lengths uniform over [ctx_lo, ctx_hi]: one draw from each of `batch` equal parts of the range, in
    random order, so that every seed has other lengths and nearly the same total."""
    rng = np.random.default_rng(seed)
    n, lo, hi = case["batch"], case["ctx_lo"], case["ctx_hi"]
    u = (rng.permutation(n) + rng.random(n)) / n
    return np.minimum(hi, lo + np.floor(u * (hi - lo + 1))).astype(np.int64)


def _matrices(case):
    """{name: (N, K, stream, sigma)} of the placed matrices; norms are separate."""
    kind = case["kind"]
    if kind == "proj":
        return {"w%d" % i: (n, k, 100 + i, 0.02) for i, (n, k) in enumerate(_shapes(case))}
    D = _dims(case)
    got = {"embed": (D.vocab, D.d, 90, 1.0)}
    if kind in ("head", "step"):
        got["lm_head"] = (D.vocab, D.d, 91, 0.02)
    use = {"qkvo": ("qkv", "o"), "mlp": ("gate_up", "down"), "step": ("qkv", "o", "gate_up", "down"), "head": ()}[kind]
    for l in range(D.layers):
        for i, (name, n, k) in enumerate(D.shapes()):
            if name in use:
                got["%s.%d" % (name, l)] = (n, k, 100 + 10 * l + i, 0.02)
    return got


def _norms(case, seed):
    D = _dims(case)
    names = ["norm_f"] + ["norm%d.%d" % (j, l) for l in range(D.layers) for j in (1, 2)]
    return {k: (1 + 0.1 * _normal(seed, 50 + i, (D.d,)).float()).to(torch.bfloat16) for i, k in enumerate(names)}


def _tokens(case, seed):
    rows = _dims(case).vocab
    return np.random.default_rng(seed + 77).integers(0, rows, size=case["batch"]).astype(np.int32)


def _kv(case, seed, layer, tokens):
    return [_normal(seed, 500 + 2 * layer + j, (tokens, case["kv_heads"], HD)) for j in (0, 1)]


# --------------------------------------------------------------------------------------------- prepare
_CTX = None


def _ctx():
    global _CTX
    if _CTX is None:
        _CTX = bd.boost_init(torch.cuda.current_device())
    return _CTX


class State:
    """The handles and device buffers of one case; what the library placed is given back with it."""

    def __init__(self):
        self.mats, self.pool = {}, None

    def place(self, case, seed):
        for name, (n, k, stream, sigma) in _matrices(case).items():
            w = _normal(seed, stream, (n, k), sigma)
            # placement copies, on the null stream, what torch's stream has written
            torch.cuda.current_stream().synchronize()
            if case["modulus"]:
                self.mats[name] = bd.boost_place_weights(_ctx(), w, n * k * 2, case["modulus"])
            else:
                pages = -(-n * k * 2 // bd.PAGE_BYTES)
                self.mats[name] = bd.boost_place_weights_map(_ctx(), w, n * k * 2, np.zeros(pages, np.uint8))

    def fill(self, case, seed, lens, cached):
        """A pool whose requests hold `lens` tokens, `cached` of them written. Each request gets the blocks of the
        first half of its context at once, as a prompt does, and the rest in turn with the others, as decoding does."""
        need = [-(-int(n) // 16) for n in lens]
        self.mb = max(need)
        layers = case.get("layers", 1)
        self.pool = bd.boost_kv_pool_create(
            _ctx(), layers, case["kv_heads"], HD, sum(need), case["modulus"] or 2,
            bd.KV_LPP if case["modulus"] else bd.KV_ALL_HBM, q_heads=case["q_heads"], max_batch=case["batch"],
            max_blocks_per_seq=self.mb)
        rows = [[] for _ in need]
        for b, n in enumerate(need):
            rows[b] += bd.boost_kv_alloc(self.pool, b, (n + 1) // 2)
        for i in range(self.mb):
            for b, n in enumerate(need):
                if len(rows[b]) < n and i % 4 == 0:
                    rows[b] += bd.boost_kv_alloc(self.pool, b, min(4, n - len(rows[b])))
        tables = np.full((len(need), self.mb), -1, np.int32)
        slots = []
        for b, r in enumerate(rows):
            tables[b, :len(r)] = r
            t = np.arange(int(cached[b]))
            slots.append(tables[b, t // 16] * 16 + t % 16)
        slots = torch.from_numpy(np.concatenate(slots).astype(np.int32)).cuda()
        for l in range(layers):
            if slots.numel():
                k, v = _kv(case, seed, l, slots.numel())
                bd.boost_kv_write(_ctx(), self.pool, l, slots, k, v, slots.numel(), _stream())
        self.tables = torch.from_numpy(tables).cuda()
        self.lens = torch.from_numpy(lens.astype(np.int32)).cuda()
        self.pos = self.lens - 1
        torch.cuda.synchronize()

    def __del__(self):
        try:
            torch.cuda.synchronize()
            for t in self.mats.values():
                bd.boost_tensor_free(t)
            if self.pool is not None:
                bd.boost_kv_pool_destroy(self.pool)
        except Exception:  # the interpreter is going down
            pass


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _f32(*shape):
    return torch.empty(shape, dtype=torch.float32, device="cuda")


def _bf16(*shape):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda")


def prepare(case, seed):
    s = State()
    s.case, kind, B = case, case["kind"], case["batch"]
    s.place(case, seed) if kind != "attn" else None
    if kind == "proj":
        s.calls = []
        for i, (n, k) in enumerate(_shapes(case)):
            s.calls.append((s.mats["w%d" % i], n, k, _normal(seed, 200 + i, (B, k)),
                            _bf16(B, n) if case["out"] == "bf16" else _f32(B, n)))
        return s
    if kind == "attn":
        lens = _lens(case, seed)
        s.fill(case, seed, lens, lens)
        s.q = _normal(seed, 200, (B, case["q_heads"], HD))
        s.o = (_bf16 if case["out"] == "bf16" else _f32)(B, case["q_heads"], HD)
        return s
    D = s.dims = _dims(case)
    s.norms = _norms(case, seed)
    s.tokens = torch.from_numpy(_tokens(case, seed)).cuda()
    if kind in ("qkvo", "step"):
        lens = _lens(case, seed)
        s.fill(case, seed, lens, lens - 1)
    if kind == "step":
        s.model = DecodeModel(_ctx(), D, B, s.mb, s.pool, s.mats, s.norms)
        return s
    s.x, s.h = _f32(B, D.d), _bf16(B, D.d)

    def slices(n, k):
        return _f32(bd.boost_gemv_slices_floats(n, k, B, bd.MAX_GEMV_SLICES))

    if kind == "qkvo":
        s.qkv_n = (D.hq + 2 * D.hkv) * HD
        s.qkv, s.sl = slices(s.qkv_n, D.d), slices(D.d, D.hq * HD)
        s.q, s.o = _bf16(B, D.hq, HD), _bf16(B, D.hq, HD)
    elif kind == "mlp":
        s.gu, s.act, s.sl = _f32(B, 2 * D.ffn), _bf16(B, D.ffn), slices(D.d, D.ffn)
    else:
        s.logits, s.ids = _f32(B, D.vocab), torch.empty((B,), dtype=torch.int32, device="cuda")
    return s


# ------------------------------------------------------------------------------------------------- run
def run(s):
    case, c, st = s.case, _ctx(), _stream()
    kind, B = case["kind"], case["batch"]
    if kind == "proj":
        dt = bd.DTYPE_BF16 if case["out"] == "bf16" else bd.DTYPE_F32
        for w, n, k, x, y in s.calls:
            bd.boost_decode_gemv(c, w, n, k, x, B, y, dt, st)
        return [y for *_, y in s.calls]
    if kind == "attn":
        bd.boost_paged_attn_decode(c, s.pool, 0, s.q, B, case["q_heads"], s.tables, s.mb, s.lens, 0.0, s.o,
                                   bd.DTYPE_BF16 if case["out"] == "bf16" else bd.DTYPE_F32, st)
        return s.o
    if kind == "step":
        ids, logits = s.model.step(s.tokens, s.pos, s.lens, s.tables, st)
        return logits
    D = s.dims
    bd.boost_embed_gather(c, s.mats["embed"], D.vocab, D.d, s.tokens, B, s.x, st)
    if kind == "qkvo":
        bd.boost_rmsnorm(c, s.x, s.norms["norm1.0"], B, D.d, EPS, s.h, st)
        n = bd.boost_decode_gemv_slices(c, s.mats["qkv.0"], s.qkv_n, D.d, s.h, B, s.qkv, bd.MAX_GEMV_SLICES, st)
        bd.boost_rope_kv_append_slices(c, s.pool, 0, s.qkv, n, D.d, s.pos, B, D.hq, THETA, s.tables, s.mb, s.q, st)
        bd.boost_paged_attn_decode(c, s.pool, 0, s.q, B, D.hq, s.tables, s.mb, s.lens, 0.0, s.o, bd.DTYPE_BF16, st)
        n = bd.boost_decode_gemv_slices(c, s.mats["o.0"], D.d, D.hq * HD, s.o, B, s.sl, bd.MAX_GEMV_SLICES, st)
        bd.boost_add_rmsnorm_slices(c, s.x, s.sl, n, D.hq * HD, s.norms["norm2.0"], B, D.d, EPS, s.h, st)
        return [s.q, s.o, s.x, s.h]
    if kind == "mlp":
        bd.boost_rmsnorm(c, s.x, s.norms["norm2.0"], B, D.d, EPS, s.h, st)
        bd.boost_decode_gemv(c, s.mats["gate_up.0"], 2 * D.ffn, D.d, s.h, B, s.gu, bd.DTYPE_F32, st)
        bd.boost_silu_mul(c, s.gu, B, D.ffn, s.act, st)
        n = bd.boost_decode_gemv_slices(c, s.mats["down.0"], D.d, D.ffn, s.act, B, s.sl, bd.MAX_GEMV_SLICES, st)
        bd.boost_add_rmsnorm_slices(c, s.x, s.sl, n, D.ffn, s.norms["norm_f"], B, D.d, EPS, s.h, st)
        return [s.gu, s.act, s.x, s.h]
    bd.boost_rmsnorm(c, s.x, s.norms["norm_f"], B, D.d, EPS, s.h, st)
    bd.boost_decode_gemv(c, s.mats["lm_head"], D.vocab, D.d, s.h, B, s.logits, bd.DTYPE_F32, st)
    bd.boost_argmax(c, s.logits, B, D.vocab, s.ids, st)
    return [s.h, s.logits, s.ids]


# ---------------------------------------------------------------------------------- work and tolerance
def work(case):
    kind, B = case["kind"], case["batch"]
    out = 2 if case.get("out") == "bf16" else 4
    nbytes = flops = 0

    def matrix(n, k, x_in=True, y_out=True):
        nonlocal nbytes, flops
        nbytes += n * k * 2 + (B * k * 2 if x_in else 0) + (B * n * out if y_out else 0)
        flops += 2 * n * k * B

    if kind == "proj":
        for n, k in _shapes(case):
            matrix(n, k)
        return {"bytes": nbytes, "flops": flops}
    if kind in ("attn", "qkvo", "step"):
        tokens = B * (case["ctx_lo"] + case["ctx_hi"]) / 2 * case.get("layers", 1)
        nbytes += tokens * case["kv_heads"] * HD * 4
        flops += tokens * case["q_heads"] * HD * 4
        if kind == "attn":
            nbytes += B * case["q_heads"] * HD * (2 + out)
            return {"bytes": nbytes, "flops": flops}
    D = _dims(case)
    for name, (n, k, _, _) in _matrices(case).items():
        if name == "embed":
            nbytes += B * k * 2
        else:  # what passes between the calls of a pass need not reach memory
            matrix(n, k, False, False)
    if kind == "qkvo":
        nbytes += B * (D.hq * HD * 4 + D.d * 6)
    elif kind == "mlp":
        nbytes += B * (D.ffn * 10 + D.d * 6)
    else:
        nbytes += B * D.vocab * 4 + (B * D.d * 2 if kind == "head" else 0)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the sums in another order (the same values in 64 bits) show: 5e-7 for 32-bit results,
    rounding flips of single values (2^-7 of the value at most) where results or operands are bf16."""
    kind = case["kind"]
    if kind in ("proj", "attn"):
        return {"rel": 1e-3, "max": 8e-3} if case["out"] == "bf16" else {"rel": 3e-6, "max": 3e-5}
    if kind == "head":
        return {"rel": 1e-3, "max": 1e-2}
    if kind == "step":  # flips in one layer travel through the next: 3e-3 seen over two layers
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 3e-3, "max": 3e-2}


# ----------------------------------------------------------------------------------------------- exact
def _round(t):
    """What a bf16 operand holds of a 64-bit value."""
    return t.to(torch.bfloat16).double()


def _times(x, w):
    """x [B, K] in 64 bits times the rows of w [N, K], some rows at a time."""
    rows = max(1, (1 << 28) // w.shape[1])
    return torch.cat([x @ w[i:i + rows].double().t() for i in range(0, w.shape[0], rows)], 1)


def _attention(case, q, k, v, lens):
    """q [B, Hq, D], k and v [sum of lens, H, D] in request order."""
    G = case["q_heads"] // case["kv_heads"]
    out, at = torch.zeros_like(q), 0
    for b, n in enumerate(int(n) for n in lens):
        kb, vb = k[at:at + n].double(), v[at:at + n].double()
        for h in range(case["kv_heads"]):
            p = torch.softmax(q[b, h * G:(h + 1) * G] @ kb[:, h].t() / math.sqrt(HD), 1)
            out[b, h * G:(h + 1) * G] = p @ vb[:, h]
        at += n
    return out


def _norm(x, w):
    return _round(x / torch.sqrt((x * x).mean(1, keepdim=True) + EPS) * w.double())


def _rope(t, pos):
    half = HD // 2
    ang = pos.double()[:, None] * THETA ** (-torch.arange(half, device="cuda", dtype=torch.float64) * 2 / HD)
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = t[..., :half], t[..., half:]
    return torch.cat([a * cos - b * sin, a * sin + b * cos], -1)


def _with_new(cached, new, lens):
    """The cached rows of every request with its new token's row after them."""
    got, at = [], 0
    for b, n in enumerate(int(n) - 1 for n in lens):
        got += [cached[at:at + n], new[b:b + 1].to(torch.bfloat16)]
        at += n
    return torch.cat(got)


def exact(case, seed):
    kind, B = case["kind"], case["batch"]
    mats = _matrices(case) if kind != "attn" else {}

    def w(name):
        n, k, stream, sigma = mats[name]
        return _normal(seed, stream, (n, k), sigma)

    if kind == "proj":
        return [_times(_normal(seed, 200 + i, (B, k)).double(), w("w%d" % i)) for i, (n, k) in enumerate(_shapes(case))]
    lens = _lens(case, seed) if kind in ("attn", "qkvo", "step") else None
    if kind == "attn":
        k, v = _kv(case, seed, 0, int(lens.sum()))
        return _attention(case, _normal(seed, 200, (B, case["q_heads"], HD)).double(), k, v, lens)
    D, norms = _dims(case), _norms(case, seed)
    x = w("embed")[torch.from_numpy(_tokens(case, seed)).cuda().long()].double()

    def attend(x, l):
        qkv = _times(_norm(x, norms["norm1.%d" % l]), w("qkv.%d" % l)).view(B, -1, HD)
        pos = torch.from_numpy(lens - 1).cuda()
        q = _round(_rope(qkv[:, :D.hq], pos))
        new = _round(_rope(qkv[:, D.hq:D.hq + D.hkv], pos)), _round(qkv[:, D.hq + D.hkv:])
        k, v = (_with_new(c, n, lens) for c, n in zip(_kv(case, seed, l, int(lens.sum()) - B), new))
        o = _round(_attention(case, q, k, v, lens))
        return q, o, x + _times(o.view(B, -1), w("o.%d" % l))

    def mlp(x, l):
        gu = _times(_norm(x, norms["norm2.%d" % l]), w("gate_up.%d" % l))
        g, u = gu[:, :D.ffn], gu[:, D.ffn:]
        act = _round(g * torch.sigmoid(g) * u)
        return gu, act, x + _times(act, w("down.%d" % l))

    if kind == "qkvo":
        q, o, x = attend(x, 0)
        return [q, o, x, _norm(x, norms["norm2.0"])]
    if kind == "mlp":
        gu, act, x = mlp(x, 0)
        return [gu, act, x, _norm(x, norms["norm_f"])]
    if kind == "step":
        for l in range(D.layers):
            x = mlp(attend(x, l)[2], l)[2]
    h = _norm(x, norms["norm_f"])
    logits = _times(h, w("lm_head"))
    return logits if kind == "step" else [h, logits, None]
