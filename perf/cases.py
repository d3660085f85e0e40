"""Performance cases of the attention path: the calls a video-diffusion
program makes through ``paper_2609_35110_amd.sol``, one case per entry point
and size class.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges,
``prepare`` builds what a program holds before the call (inputs from the seed
alone, the rotary table, norm weights, workspaces, cached reference keys),
``run`` is one pass through the public entry points, ``work`` the bytes and
operations a pass cannot do without, ``tolerance`` how far another correct
implementation may be off, ``exact`` the same outputs in 64 bits from plain
torch.

A case's keys: ``kind`` (below), B, H, the latent grid T x Hl x Wl, ``text``
(unrotated tokens ahead of the video tokens), and per kind ``norm`` (QK
normalisation), ``boost`` (1 % of the keys times 8: peaked rows), ``ref``
(frames of a cached reference video ahead of the own keys), ``tau`` (routing
threshold), ``fmt`` (0 bf16, 1 E4M3, 2 block-INT8 output records), ``split``
(partial rotary split).

  fwd      attn_fwd: the workspace-free call
  ws       attn_fwd_ws: prepare and attend on a workspace the program keeps
  layer    prepare_kv_ex + attn_fwd_prepared_ex: one layer of a denoising step
  sparse   prepare_kv_ex + sparse_route + attn_fwd_sparse
  prepare  prepare_kv_ex of a reference segment into a longer key sequence
  encode   qkv_encode_packed: the sender's side of the quantised QKV exchange
  decode   qkv_decode: its other side, for a consumer that wants bf16 tensors
  records  prepare_kv_records + attn_fwd_records: the receiver's attention
  rope     qknorm_rope3d / rope3d: the standalone normalisation and rotation
"""
import math

import torch

from paper_2609_35110_amd import sol

D = 128
EPS = 1e-6
QB, KB = sol.SPARSE_QUERY_BLOCK, sol.SPARSE_KEY_BLOCK
REC, OUT_REC = sol.QKV_RECORD_BYTES, sol.OUT_RECORD_BYTES
MAX_FLOPS = 4.0 * 111600 ** 2 * D * 40  # the largest listed case
MAX_VALUES = 40 * 111600 * D            # of one of its tensors
EXACT_FLOPS = 1e14                      # above this a 64-bit evaluation takes too long


def case(kind, B, H, T, Hl, Wl, text=0, **kw):
    c = {"kind": kind, "B": B, "H": H, "T": T, "Hl": Hl, "Wl": Wl, "text": text}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: the smoke test's grid, bound by latency
        case("fwd", 1, 2, 3, 8, 8, name="fwd tiny"),
        # the low-resolution stage's layer through the call without a workspace
        case("fwd", 1, 24, 8, 30, 52, name="fwd low"),
        # one of eight GPUs' head share of that layer: fewer query tiles than CUs
        case("ws", 1, 3, 8, 30, 52, name="ws low share"),
        # the same layer whole, keys cached for one reference video, E4M3 for the next GEMM
        case("layer", 1, 24, 8, 30, 52, text=512, ref=8, fmt=1, name="layer low ref"),
        # 480p with peaked rows (the second pass of the attention)
        case("layer", 1, 40, 31, 30, 52, boost=True, name="layer p480"),
        # 720p, the whole layer: the headline size
        case("layer", 1, 40, 31, 45, 80, name="layer p720"),
        # one GPU's head share of the 720p layer: text prefix, QK norm, batch 2
        case("layer", 2, 5, 31, 45, 80, text=512, norm=True, name="layer share"),
        # block-sparse 720p refinement step
        case("sparse", 1, 40, 31, 45, 80, tau=1.25, name="sparse p720"),
        # a reference video's keys written once into the step's key sequence
        case("prepare", 1, 40, 8, 45, 80, norm=True, tail=1001, name="prepare ref"),
        # the sender: four of the 720p latent's frames, every head, packed QKV
        case("encode", 1, 40, 4, 45, 80, norm=True, name="encode shard"),
        # the receiver: one GPU's heads, attention from records
        case("records", 1, 5, 31, 30, 52, fmt=0, name="records share"),
        # a reference video's queries normalised and rotated on their own
        case("rope", 1, 40, 8, 45, 80, norm=True, name="rope ref"),
    ]


def tokens(c):
    return c["text"] + c["T"] * c["Hl"] * c["Wl"]


def n_ref(c):
    return c.get("ref", 0) * c["Hl"] * c["Wl"]


def attention_flops(c):
    N = tokens(c)
    return 4.0 * c["B"] * c["H"] * N * (N + n_ref(c)) * D


KINDS = ("fwd", "ws", "layer", "layer", "sparse", "prepare", "encode", "decode", "records", "rope")
ATTENTION = ("fwd", "ws", "layer", "sparse", "records")
SPLITS = ("", "", "", "16/24/24", "0/64/64", "8/8/8")


def draw(rng):
    """One more case: any kind, heads 1 to 40, grids 1x8x8 to 31x45x80, odd
    and ragged ones among them, options at random."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(KINDS)
        c = case(kind, rng.choice((1, 1, 2)), rng.choice((1, 2, 3, 5, 10, 12, 24, 40)), log_int(1, 31),
                 log_int(8, 45), log_int(8, 80), text=rng.choice((0, 0, rng.randint(1, 512))))
        if kind == "layer":
            c.update(norm=rng.random() < 0.5, boost=rng.random() < 0.25, fmt=rng.choice((0, 0, 1, 2)),
                     ref=rng.choice((0, 0, 1, 8)), split=rng.choice(SPLITS))
        elif kind == "sparse":
            c.update(tau=rng.choice((1.0, 1.25, 1.5)))
        elif kind == "prepare":
            c.update(norm=rng.random() < 0.5, tail=rng.randint(0, 2000), split=rng.choice(SPLITS))
        elif kind in ("encode", "rope"):
            c.update(norm=rng.random() < 0.5)
        elif kind == "records":
            c.update(fmt=rng.choice((0, 0, 1, 2)))
        N = tokens(c)
        if c["B"] * c["H"] * (N + n_ref(c) + c.get("tail", 0)) * D > MAX_VALUES:
            continue
        if kind in ATTENTION and attention_flops(c) > MAX_FLOPS:
            continue
        if kind == "sparse" and N < 2000:
            continue  # a few key blocks are not worth a routing
        return c


# ------------------------------------------------------------------- inputs

def generator(seed):
    return torch.Generator("cuda").manual_seed(seed)


def randn(gen, *shape):
    """N(0, 1) in bf16, drawn slab by slab so that no fp32 copy of a large tensor exists."""
    x = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    rows = x.view(-1, shape[-1])
    step = 1 << 21
    for a in range(0, rows.shape[0], step):
        part = rows[a:a + step]
        part.copy_(torch.randn(part.shape, generator=gen, device="cuda"))
    return x


def split_of(c):
    return tuple(int(x) for x in c["split"].split("/")) if c.get("split") else None


def row_scales(gen, x):
    """Rows times 2^e, e in [-4, 4]: what a projection hands to the QK normalisation."""
    e = torch.randint(-4, 5, x.shape[:-1] + (1,), generator=gen, device="cuda")
    return x.mul_(torch.exp2(e.float()).to(torch.bfloat16))


def prepare(c, seed):
    gen = generator(seed)
    B, H, N, kind = c["B"], c["H"], tokens(c), c["kind"]
    grid = (c["T"], c["Hl"], c["Wl"])
    s = {"c": c, "grid": grid, "split": split_of(c)}
    s["table"] = sol.rope3d_table(*grid, split=s["split"])
    if c.get("norm"):
        for name in ("q_gamma", "k_gamma"):
            s[name] = 1 + 0.25 * torch.randn(D, generator=gen, device="cuda")
    if kind == "encode":
        s["qkv"] = randn(gen, B, N, 3, H, D)
        if c.get("norm"):
            row_scales(gen, s["qkv"][:, :, :2])
        s["rec"] = torch.empty((B, N, H, REC), dtype=torch.uint8, device="cuda")
        return s
    q, k, v = (randn(gen, B, H, N, D) for _ in range(3))
    if kind == "sparse":  # a per-head direction shared by q and k: local attention
        shared = torch.randn((B, H, 1, D), generator=gen, device="cuda").to(torch.bfloat16)
        q += shared
        k += shared
    if c.get("norm"):
        row_scales(gen, q)
        row_scales(gen, k)
    if c.get("boost"):
        at = torch.randperm(N, generator=gen, device="cuda")[:N // 100]
        k[:, :, at] = k[:, :, at] * 8
    s.update(q=q, k=k, v=v)
    if kind in ("decode", "records"):
        s["rec"] = sol.qkv_encode(q, k, v, *grid, s["table"])
        del s["q"], s["k"], s["v"]
    if kind == "prepare":
        s["n_kv"] = N + c["tail"]
        s["prep"] = sol.prepared_kv_buffers(B, H, s["n_kv"], "cuda")
        del s["q"]
    if kind == "rope":
        s["x"], s["y"] = q, torch.empty_like(q)
        del s["q"], s["k"], s["v"]
    if kind in ("layer", "sparse", "records"):
        s["n_kv"] = N + n_ref(c)
        s["prep"] = sol.prepared_kv_buffers(B, H, s["n_kv"], "cuda")
    if n_ref(c):  # the reference video's keys and values, cached at the first step
        rgrid = (c["ref"], c["Hl"], c["Wl"])
        s["rk"], s["rv"] = randn(gen, B, H, n_ref(c), D), randn(gen, B, H, n_ref(c), D)
        s["rgrid"] = rgrid
        sol.prepare_kv_ex(s["rk"], s["rv"], *rgrid, sol.rope3d_table(*rgrid, split=s["split"]), *s["prep"], 0,
                          s["n_kv"], s.get("k_gamma"), EPS, s["split"])
    if kind == "ws":
        s["workspace"] = sol.attn_workspace(q)
    if kind == "sparse":
        s["workspace"] = sol.sparse_workspace(q).zero_()
    if kind in ATTENTION:
        fmt = c.get("fmt", 0)
        s["out"] = (torch.empty((B, H, N, D), dtype=torch.bfloat16, device="cuda") if fmt == 0 else
                    torch.empty((B, H, N, D), dtype=torch.uint8, device="cuda") if fmt == 1 else
                    torch.empty((B, N, H, OUT_REC), dtype=torch.uint8, device="cuda"))
    return s


# --------------------------------------------------------------------- runs

def run(s):
    c, grid, kind = s["c"], s["grid"], s["c"]["kind"]
    fmt = c.get("fmt", 0)
    how = {"out": s.get("out"), "fp8": fmt == 1, "int8_records": fmt == 2}
    if kind == "fwd":
        return sol.attn_fwd(s["q"], s["k"], s["v"], *grid, s["table"], out=s["out"])
    if kind == "ws":
        return sol.attn_fwd_ws(s["q"], s["k"], s["v"], *grid, s["table"], workspace=s["workspace"], out=s["out"])
    if kind == "layer":
        sol.prepare_kv_ex(s["k"], s["v"], *grid, s["table"], *s["prep"], s["n_kv"] - tokens(c), s["n_kv"],
                          s.get("k_gamma"), EPS, s["split"])
        return sol.attn_fwd_prepared_ex(s["q"], *s["prep"], s["n_kv"], *grid, s["table"], s.get("q_gamma"), EPS,
                                        split=s["split"], **how)
    if kind == "sparse":
        sol.prepare_kv_ex(s["k"], s["v"], *grid, s["table"], *s["prep"])
        sol.sparse_route(s["q"], s["prep"][0], *grid, s["table"], c["tau"], s["workspace"])
        out = sol.attn_fwd_sparse(s["q"], *s["prep"], *grid, s["table"], s["workspace"], out=s["out"])
        counts, _ = sol.sparse_routing(s["workspace"], c["B"], c["H"], tokens(c))
        return {"out": out, "counts": counts}
    if kind == "prepare":
        return sol.prepare_kv_ex(s["k"], s["v"], *grid, s["table"], *s["prep"], 0, s["n_kv"], s.get("k_gamma"), EPS,
                                 s["split"])
    if kind == "encode":
        return sol.qkv_encode_packed(s["qkv"], *grid, s["table"], s.get("q_gamma"), s.get("k_gamma"), EPS, s["rec"])
    if kind == "decode":
        return sol.qkv_decode(s["rec"])
    if kind == "records":
        sol.prepare_kv_records(s["rec"], *s["prep"])
        return sol.attn_fwd_records(s["rec"], *s["prep"], **how)
    if c.get("norm"):
        return sol.qknorm_rope3d(s["x"], *grid, s["table"], s["q_gamma"], EPS, out=s["y"])
    return sol.rope3d(s["x"], *grid, s["table"], out=s["y"])


def sparse_density(c):
    """Share of (query, key) pairs that the routing keeps on these inputs (measured at 720p)."""
    return {1.0: 0.169, 1.25: 0.124, 1.5: 0.087}[c["tau"]]


def work(c):
    """One pass: every input read once, every output written once; the two
    products of the attention.  Prepared keys are an output of the calls that
    make them; the attention reads them from there."""
    kind, N = c["kind"], tokens(c)
    rows = c["B"] * c["H"] * N
    row = 2 * D
    out_row = (row, D, OUT_REC)[c.get("fmt", 0)]
    if kind in ("fwd", "ws"):
        return {"bytes": rows * 4 * row, "flops": attention_flops(c)}
    if kind == "layer":
        keys = c["B"] * c["H"] * (N + n_ref(c))
        return {"bytes": rows * (3 * row + 2 * row + out_row) + keys * 2 * row, "flops": attention_flops(c)}
    if kind == "sparse":
        return {"bytes": rows * (3 * row + 2 * row + 2 * row + row),
                "flops": attention_flops(c) * sparse_density(c)}
    if kind == "prepare":
        return {"bytes": rows * 4 * row, "flops": 0}
    if kind == "encode":
        return {"bytes": rows * (3 * row + REC), "flops": 0}
    if kind == "decode":
        return {"bytes": rows * (3 * row + REC), "flops": 0}
    if kind == "records":
        return {"bytes": rows * (REC + 2 * row + 2 * row + out_row), "flops": attention_flops(c)}
    return {"bytes": rows * 2 * row, "flops": 0}


def tolerance(c):
    """bf16 attention outputs: the rounding of the output and of the fp16
    probabilities leaves 1.7e-3 against 64 bits (2-norm), here four times
    that.  Quantised attention outputs: a code changes where the value sits
    within that error of a rounding midpoint.  Records and rotations without
    normalisation round exactly once from an exact value; with it a bf16
    rounding may fall the other way (a 2^-8 step on few values)."""
    kind = c["kind"]
    if kind in ATTENTION:
        return {"rel": 7e-3, "max": 0.05, "differ": 1e-2}
    if kind in ("encode", "decode") or not c.get("norm"):
        return "exact"
    return {"rel": 1e-3, "max": 0.02}


# ------------------------------------------------------------- in 64 bits

def rotate(x, c, grid, split, gamma=None):
    """bf16 of the exact normalisation and rotation of x [..., N, D], as the
    contract rounds it, in float64."""
    x = x.double()
    if gamma is not None:
        x = x / torch.sqrt(x.square().mean(-1, keepdim=True) + EPS) * gamma.double()
    T, Hl, Wl = grid
    n = x.shape[-2]
    text = n - T * Hl * Wl
    i = torch.arange(T * Hl * Wl, device=x.device)
    pos = (i // (Hl * Wl), i // Wl % Hl, i % Wl)
    d0 = 0
    out = x.clone()
    for p, d in zip(pos, split or sol.DEFAULT_SPLIT):
        if d == 0:
            continue
        freq = torch.pow(torch.tensor(10000.0, dtype=torch.float64, device=x.device),
                         -torch.arange(0, d, 2, dtype=torch.float64, device=x.device) / d)
        a = p.double()[:, None] * freq
        cos, sin = a.cos(), a.sin()
        u, w = x[..., text:, d0:d0 + d:2], x[..., text:, d0 + 1:d0 + d:2]
        out[..., text:, d0:d0 + d:2] = u * cos - w * sin
        out[..., text:, d0 + 1:d0 + d:2] = u * sin + w * cos
        d0 += d
    return out.bfloat16().double()


def attend(q, k, v, mask=None):
    """softmax(q k^T / sqrt(D)) v of one slab in float64, in bands of query rows."""
    out = torch.empty_like(q)
    kt = k.t().contiguous()
    step = QB * max(1, (1 << 28) // (QB * k.shape[0]))
    for a in range(0, q.shape[0], step):
        p = q[a:a + step] @ kt
        p *= D ** -0.5
        if mask is not None:
            m = mask[a // QB:-(-(a + p.shape[0]) // QB)].repeat_interleave(QB, 0)[:p.shape[0]]
            p.masked_fill_(~m.repeat_interleave(KB, 1)[:, :k.shape[0]], -math.inf)
        p -= p.amax(1, keepdim=True)
        p.exp_()
        out[a:a + step] = (p @ v) / p.sum(1, keepdim=True)
    return out


def pooled(x, block):
    n = x.shape[0]
    full = n // block * block
    parts = [x[:full].view(-1, block, D).mean(1)] if full else []
    if full < n:
        parts.append(x[full:].mean(0, keepdim=True))
    return torch.cat(parts)


def kept_blocks(q, k, text, tau):
    """The routing of one slab: key blocks over mean + tau std, prefix blocks, the best block."""
    s = pooled(q, QB) @ pooled(k, KB).t().contiguous() * D ** -0.5
    keep = s > s.mean(1, keepdim=True) + tau * s.std(1, correction=0, keepdim=True)
    keep[torch.arange(s.shape[0], device=s.device), s.argmax(1)] = True
    keep[:, :-(-text // KB)] = True
    keep[:-(-text // QB)] = True
    return keep


def decoded(rec):
    """q, k, v of block-INT8 records in float64 (codes times scales, rounded to bf16)."""
    B, N, H = rec.shape[:3]
    codes = rec[..., :384].view(torch.int8).double().view(B, N, H, 3, 4, 32)
    e = rec[..., 384:396].int().view(B, N, H, 3, 4)
    m, x = (e & 7).double(), e >> 3
    scale = torch.where(x == 0, m * 2.0 ** -17, (1 + m / 8) * torch.exp2((x - 15).double()))
    val = (codes * scale[..., None]).bfloat16().view(B, N, H, 3, D)
    return [val[:, :, :, p].transpose(1, 2).contiguous() for p in range(3)]


def exact(c, seed):
    kind = c["kind"]
    if kind in ATTENTION and (attention_flops(c) > EXACT_FLOPS or c.get("fmt", 0)):
        return None  # too long, or codes
    if kind == "encode":
        return None
    s = prepare(c, seed)
    B, H, N = c["B"], c["H"], tokens(c)
    grid, split = s["grid"], s["split"]
    if kind == "decode":
        return tuple(decoded(s["rec"]))
    if kind == "rope":
        out = torch.empty((B, H, N, D), dtype=torch.float64, device="cuda")
        for b in range(B):
            for h in range(H):
                out[b, h] = rotate(s["x"][b, h], c, grid, split, s.get("q_gamma"))
        return out
    if kind == "prepare":
        tiles = -(-s["n_kv"] // 32)
        kt = torch.zeros((B * H, tiles, 8, 2, 32, 8), dtype=torch.float64, device="cuda")
        vt = torch.zeros((B * H, tiles, 2, 4, 2, 32, 8), dtype=torch.float64, device="cuda")
        for b in range(B):
            for h in range(H):
                k = torch.zeros((tiles * 32, D), dtype=torch.float64, device="cuda")
                v = torch.zeros_like(k)
                k[:N] = rotate(s["k"][b, h], c, grid, split, s.get("k_gamma"))
                v[:N] = s["v"][b, h].double()
                # K: [kk][half][key][8 dims];  V: [kst][db][half][dim][4 + 4 keys]
                kt[b * H + h] = k.view(tiles, 32, 8, 2, 8).permute(0, 2, 3, 1, 4)
                vt[b * H + h] = v.view(tiles, 2, 2, 2, 4, 4, 32).permute(0, 1, 5, 3, 6, 2, 4).reshape(
                    tiles, 2, 4, 2, 32, 8)
        return kt.view(-1), vt.view(-1)
    if kind == "records":
        q, k, v = decoded(s["rec"])
    out = torch.empty((B, H, N, D), dtype=torch.float64, device="cuda")
    for b in range(B):
        for h in range(H):
            mask = None
            if kind == "records":
                qh, kh, vh = (x[b, h].double() for x in (q, k, v))
            else:
                qh = rotate(s["q"][b, h], c, grid, split, s.get("q_gamma"))
                kh = rotate(s["k"][b, h], c, grid, split, s.get("k_gamma"))
                vh = s["v"][b, h].double()
                if n_ref(c):
                    kh = torch.cat([rotate(s["rk"][b, h], c, s["rgrid"], split, s.get("k_gamma")), kh])
                    vh = torch.cat([s["rv"][b, h].double(), vh])
            if kind == "sparse":
                mask = kept_blocks(qh, kh, c["text"], c["tau"])
            out[b, h] = attend(qh, kh, vh, mask)
    return {"out": out, "counts": None} if kind == "sparse" else out
