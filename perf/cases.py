"""Performance cases of the ReKV path: what a program that uses this library has it do.

Three kinds of call sequence, each through the public binding (`paper_2503_00540_amd.rekv.Rekv`):

* encode - new video tokens: windowed attention over n_chunks chunks, then the new frames' vectors;
* answer - a question arrives: retrieval, reload of the retrieved KV (or attention that reads it in
  place), question attention;
* decode - one answer token (or a few drafted ones) over the retrieved KV and the text so far.

A case is a dict of plain values.  `listed()` names the ones that stand for the benchmark's
configurations and the sizes around them; `draw()` gives more of the same ranges.  Inputs follow the
benchmark's recipe (N(0,1) plus a per-frame offset of sigma 0.5; question queries near the key offsets
of three planted frames) drawn on the GPU from the seed.
"""
from __future__ import annotations

import math

import torch

from paper_2503_00540_amd.rekv import Rekv

DEV = "cuda:0"
PLANTED = 3              # frames a question is near


# ----------------------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------------------
def _heads(hq, hkv, d, dtype="bf16"):
    return {"hq": hq, "hkv": hkv, "d": d, "dtype": dtype}


H_TINY = _heads(4, 1, 64, "f32")          # the tiny fp32 configuration
H_05B = _heads(14, 2, 64)                 # 0.5B-class decoder
H_7B = _heads(28, 4, 128)                 # 7B-class decoder
H_72B = _heads(64, 8, 128)                # 72B-class decoder


def _encode(heads, nf, chunk_frames, window_frames, past_frames, n_chunks, **kw):
    return {"kind": "encode", **heads, "nf": nf, "chunk_frames": chunk_frames, "window_frames": window_frames,
            "past_frames": past_frames, "n_chunks": n_chunks, **kw}


def _answer(heads, nf, frames, questions, q_tokens, top_k, context, layers=1, block=1, external_dim=0, **kw):
    return {"kind": "answer", **heads, "nf": nf, "frames": frames, "questions": questions, "q_tokens": q_tokens,
            "top_k": top_k, "context": context, "layers": layers, "block": block, "external_dim": external_dim, **kw}


def _decode(heads, nf, questions, top_k, text_tokens, new_tokens, no_alloc, **kw):
    return {"kind": "decode", **heads, "nf": nf, "questions": questions, "top_k": top_k, "text_tokens": text_tokens,
            "new_tokens": new_tokens, "no_alloc": no_alloc, **kw}


def listed():
    return [
        # the tiny fp32 stream, all of it: fp32 exists for accuracy work at sizes like this
        dict(_encode(H_TINY, 16, 1, 4, 0, 32), name="encode_f32_tiny"),
        # a live stream, one frame at a time, window full: what arrives at every frame of every layer
        dict(_encode(H_05B, 196, 1, 16, 40, 1), name="live_frame_05b"),
        dict(_encode(H_7B, 196, 1, 16, 100, 1), name="live_frame_7b"),
        # a recorded stream in one call: 256 frames (the benchmark's headline), and the 28-layer
        # configuration's layer (1,024 frames in four-frame chunks, window 32 frames) - the largest
        dict(_encode(H_7B, 196, 1, 16, 0, 256), name="recorded_256f_7b"),
        dict(_encode(H_7B, 196, 4, 32, 0, 256), name="recorded_1024f_7b"),
        # a single question on a short stream, KV in HBM
        dict(_answer(H_7B, 196, 256, 1, 32, 16, "gather"), name="question_7b"),
        # an hour at 0.5 FPS, KV offloaded to pinned host memory
        dict(_answer(H_7B, 196, 1800, 1, 64, 64, "host"), name="question_hour_host"),
        # 64 users asking at once about one 72B-class stream
        dict(_answer(H_72B, 144, 2048, 64, 32, 32, "gather"), name="questions_64_72b"),
        # one question through all 28 layers, each with its own table and selection
        dict(_answer(H_7B, 196, 1024, 1, 48, 32, "layers", layers=28), name="question_28_layers"),
        # small decoder, block retrieval, keys re-positioned, frames read in place; ragged sizes
        dict(_answer(H_05B, 196, 777, 5, 23, 40, "inplace_rope", block=8), name="questions_blocks_05b"),
        # one answer token: one user with 64 retrieved frames, and 64 users
        dict(_decode(H_7B, 196, 1, 64, 97, 1, True), name="decode_7b"),
        dict(_decode(H_72B, 144, 64, 32, 96, 1, False), name="decode_64_72b"),
    ]


CONTEXTS = ("gather", "gather", "host", "layers", "rope", "inplace", "inplace_rope")


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    heads = rng.choice([H_05B, H_7B, H_7B, H_72B, _heads(16, 8, 64), _heads(8, 2, 128)])
    nf = rng.choice([196, 144, rng.randint(33, 256)])
    f32 = rng.random() < 0.12              # fp32 contexts stay at the sizes accuracy work uses
    if f32:
        heads = dict(rng.choice([H_TINY, H_05B]), dtype="f32")
        nf = rng.randint(8, 64)
    kind = rng.choice(["encode", "encode", "answer", "answer", "decode"])
    if kind == "encode":
        window = _log_int(rng, 2, 77)      # up to the 15K tokens of the paper's setting
        chunk = rng.choice([1, 1, 2, 3, 4])
        n_chunks = 1 if rng.random() < 0.5 else _log_int(rng, 2, 32 if f32 else 256)
        return _encode(heads, nf, chunk, min(window, 8) if f32 else window, rng.randint(0, 120), n_chunks)
    top_k = _log_int(rng, 4, 64)
    questions = 1 if rng.random() < 0.5 else _log_int(rng, 2, 4 if f32 else 64)
    if kind == "decode":
        return _decode(heads, nf, questions, min(top_k, 16) if f32 else top_k, _log_int(rng, 16, 320),
                       1 if rng.random() < 0.75 else rng.randint(2, 8), rng.random() < 0.5)
    context = rng.choice(CONTEXTS)
    frames = max(_log_int(rng, 64, 3600), top_k + 8)
    layers, block, ext = 1, 1, 0
    if context == "layers":
        layers, questions, frames = _log_int(rng, 2, 28), 1, min(frames, 1024)
    elif rng.random() < 0.3:
        block = rng.choice([2, 4, 5, 8])
    elif rng.random() < 0.2:
        ext = rng.choice([768, 1152])
    if context == "host":
        frames = min(frames, 1800)
    return _answer(heads, nf, frames, questions, rng.randint(8, 64), min(top_k, 16) if f32 else top_k, context,
                   layers=layers, block=block, external_dim=ext)


def _cost(case):
    w = work(case)
    link = 20.0 if case.get("context") == "host" else 1.0
    return max(link * w["bytes"] / 4e12, w["flops"] / (1e15 if case["dtype"] == "bf16" else 1e13))


def draw(rng):
    """One more case of the same ranges; never dearer than the largest listed one."""
    most = max(_cost(c) for c in listed())
    while True:
        case = _draw_once(rng)
        if _cost(case) <= most:
            return case


# ----------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------
def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _stream(g, frames, nf, heads, d, dtype):
    """[frames * nf, heads, d] of N(0,1) + a per-frame offset, and the offsets [frames, heads, d]."""
    out = torch.empty((frames * nf, heads, d), dtype=dtype, device=DEV)
    off = 0.5 * torch.randn((frames, 1, heads, d), device=DEV, generator=g)
    for f in range(0, frames, 256):
        f1 = min(f + 256, frames)
        x = torch.randn((f1 - f, nf, heads, d), device=DEV, generator=g) + off[f:f1]
        out[f * nf:f1 * nf] = x.reshape(-1, heads, d).to(dtype)
    return out, off[:, 0]


def _randn(g, shape, dtype):
    return torch.randn(shape, device=DEV, generator=g).to(dtype)


def _frame_table(k, frames, nf, d_prime):
    """The stream's frame vectors, as the encode side has left them in HBM when a question arrives."""
    out = torch.empty((frames, d_prime), dtype=torch.float32, device=DEV)
    for f in range(0, frames, 256):
        f1 = min(f + 256, frames)
        out[f:f1] = k[f * nf:f1 * nf].view(f1 - f, nf, d_prime).float().mean(dim=1)
    return out


def prepare(case, seed):
    c = case
    dt = _dtype(c)
    hq, hkv, d, nf = c["hq"], c["hkv"], c["d"], c["nf"]
    g = torch.Generator(device=DEV).manual_seed(seed)
    gc = torch.Generator().manual_seed(seed)
    s = {"case": c, "r": Rekv(hq, hkv, d, nf, c["dtype"])}
    if c["kind"] == "encode":
        new = c["n_chunks"] * c["chunk_frames"]
        total = c["past_frames"] + new
        s["q"], _ = _stream(g, new, nf, hq, d, dt)
        s["k"], _ = _stream(g, total, nf, hkv, d, dt)
        s["v"], _ = _stream(g, total, nf, hkv, d, dt)
        s["out"] = torch.empty_like(s["q"])
        s["table"] = torch.empty((new, hkv * d), dtype=torch.float32, device=DEV)
        s["k_new"] = s["k"][c["past_frames"] * nf:]
        return s
    nq, k = c["questions"], c["top_k"]
    if c["kind"] == "decode":
        n_text = c["text_tokens"]
        room = n_text + 32                 # the text cache has room for the tokens still to come
        s["k_ret"] = torch.empty((nq, k * nf, hkv, d), dtype=dt, device=DEV)
        s["v_ret"] = torch.empty_like(s["k_ret"])
        for i in range(nq):
            s["k_ret"][i] = _stream(g, k, nf, hkv, d, dt)[0]
            s["v_ret"][i] = _stream(g, k, nf, hkv, d, dt)[0]
        s["k_text"], s["v_text"] = _randn(g, (nq, room, hkv, d), dt), _randn(g, (nq, room, hkv, d), dt)
        s["q"] = _randn(g, (nq, c["new_tokens"], hq, d), dt)
        s["out"] = torch.empty_like(s["q"])
        s["n_sel"] = torch.full((nq,), k, dtype=torch.int32, device=DEV)
        return s
    frames, layers, nt = c["frames"], c["layers"], c["q_tokens"]
    rows = layers * nq
    s["k"], s["v"], s["tables"], qq = [], [], [], []
    for _ in range(layers):
        kk, off = _stream(g, frames, nf, hkv, d, dt)
        s["k"].append(kk)
        s["v"].append(_stream(g, frames, nf, hkv, d, dt)[0])
        s["tables"].append(_frame_table(kk, frames, nf, hkv * d))
        for _ in range(nq):                # queries near the planted frames' key offsets
            p = torch.randperm(frames, generator=gc)[:PLANTED].sort().values.to(DEV)
            base = off[p][torch.arange(nt, device=DEV) % PLANTED].repeat_interleave(hq // hkv, dim=1)
            qq.append((base + 0.3 * torch.randn((nt, hq, d), device=DEV, generator=g)).to(dt))
    s["tables"] = torch.stack(s["tables"])
    s["q"] = torch.stack(qq)
    s["k_q"], s["v_q"] = _randn(g, (rows, nt, hkv, d), dt), _randn(g, (rows, nt, hkv, d), dt)
    s["out"] = torch.empty_like(s["q"])
    if c["external_dim"]:
        s["frame_emb"] = _randn(g, (frames, c["external_dim"]), torch.float32)
        s["q_emb"] = _randn(g, (nq, c["external_dim"]), torch.float32)
    if c["context"] == "host":             # offloaded: the KV lives in pinned host memory only
        for key in ("k", "v"):
            h = torch.empty(s[key][0].shape, dtype=dt, pin_memory=True)
            h.copy_(s[key][0])
            s[key] = [h]
    n_ret = _retrieved(c)
    if c["context"] in ("gather", "host", "layers"):
        s["k_ret"] = torch.empty((rows, n_ret * nf, hkv, d), dtype=dt, device=DEV)
        s["v_ret"] = torch.empty_like(s["k_ret"])
    if c["context"] == "inplace_rope":
        s["k_pos"] = torch.empty((rows, n_ret * nf, hkv, d), dtype=dt, device=DEV)
    return s


def _retrieved(c):
    """Frames listed per question: whole blocks under block retrieval."""
    return -(-c["top_k"] // c["block"]) * c["block"]


# ----------------------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------------------
def run(s):
    c, r = s["case"], s["r"]
    nf = c["nf"]
    if c["kind"] == "encode":
        l_x = c["chunk_frames"] * nf
        r.encode_chunk(s["q"], s["k"], s["v"], c["past_frames"] * nf, l_x, c["n_chunks"], c["window_frames"] * nf, out=s["out"])
        r.frame_keys(s["k_new"], c["n_chunks"] * c["chunk_frames"], out=s["table"])
        return s["out"], s["table"]
    if c["kind"] == "decode":
        r.decode_attention(s["q"], s["k_ret"], s["v_ret"], s["k_text"], s["v_text"], c["text_tokens"], out=s["out"],
                           n_sel=s["n_sel"], no_alloc=c["no_alloc"])
        return s["out"]
    F, k = c["frames"], c["top_k"]
    # which frames
    if c["block"] > 1:
        blocks = r.block_keys(s["tables"][0], F, c["block"])
        blk, _, _ = r.retrieve_topk(blocks, blocks.shape[0], s["q"], -(-k // c["block"]))
        idx, n_sel = r.expand_blocks(blk, c["block"], F)
    elif c["external_dim"]:
        idx, n_sel, _ = r.retrieve_external(s["frame_emb"], s["q_emb"], k, tau=0.07)
    else:
        stride = F * c["hkv"] * c["d"] if c["layers"] > 1 else 0
        idx, n_sel, _ = r.retrieve_topk(s["tables"], F, s["q"], k, frame_keys_stride=stride)
    # their KV, and the question's attention
    ctx, nt = c["context"], c["q_tokens"]
    if ctx == "inplace":
        r.attention_indexed(s["q"], s["k"][0], s["v"][0], idx, idx.shape[1], s["k_q"], s["v_q"], nt, n_src_frames=F,
                            n_sel=n_sel, out=s["out"])
        return idx, n_sel, s["out"]
    if ctx == "inplace_rope":
        r.attention_indexed_rope(s["q"], s["k"][0], s["v"][0], idx, s["k_q"], s["v_q"], nt, n_src_frames=F, n_sel=n_sel,
                                 k_pos=s["k_pos"], out=s["out"])
        return idx, n_sel, s["k_pos"], s["out"]
    if ctx == "rope":
        gk, gv = r.gather_kv_rope(s["k"][0], s["v"][0], idx, n_src_frames=F)
    elif ctx == "layers":
        gk, gv = s["k_ret"], s["v_ret"]
        r.gather_kv_layers(s["k"], s["v"], idx.view(c["layers"], c["questions"], k), n_src_frames=F, dst_k=gk, dst_v=gv)
    else:
        gk, gv = r.gather_kv(s["k"][0], s["v"][0], idx, n_src_frames=F, dst_k=s["k_ret"], dst_v=s["v_ret"])
    r.qa_attention(s["q"], gk, gv, s["k_q"], s["v_q"], out=s["out"], n_sel=n_sel)
    return idx, n_sel, gk, gv, s["out"]


# ----------------------------------------------------------------------------------------
# what a pass cannot do without, and how far correct results may lie apart
# ----------------------------------------------------------------------------------------
def work(case):
    c = case
    es = 2 if c["dtype"] == "bf16" else 4
    hq, hkv, d, nf = c["hq"], c["hkv"], c["d"], c["nf"]
    kv, q = 2 * hkv * d * es, hq * d * es              # bytes of a token's K and V, of its queries
    per_pair = 4.0 * hq * d                            # FLOP per visible (query, key) pair, all heads
    if c["kind"] == "encode":
        l_x, l_l, past = c["chunk_frames"] * nf, c["window_frames"] * nf, c["past_frames"] * nf
        new = c["n_chunks"] * l_x
        pairs = sum(l_x * min(l_l, past + i * l_x) + l_x * (l_x + 1) // 2 for i in range(c["n_chunks"]))
        frames = c["n_chunks"] * c["chunk_frames"]
        return {"bytes": 2 * new * q + (min(l_l, past) + new) * kv + frames * hkv * d * 4,
                "flops": per_pair * pairs + new * hkv * d}
    nq = c["questions"]
    if c["kind"] == "decode":
        n, t, m = c["top_k"] * nf, c["text_tokens"], c["new_tokens"]
        return {"bytes": nq * ((n + t) * kv + 2 * m * q), "flops": per_pair * nq * (m * (n + t - m) + m * (m + 1) // 2)}
    F, rows, nt = c["frames"], c["layers"] * nq, c["q_tokens"]
    n_ret = _retrieved(c)
    # distinct frames the questions of a layer read between them (independent picks)
    distinct = c["layers"] * F * (1.0 - (1.0 - min(n_ret, F) / F) ** nq)
    nbytes = rows * nt * (2 * q + kv) + distinct * nf * kv + rows * n_ret * 4
    dim = c["external_dim"] or hkv * d
    nbytes += c["layers"] * F * dim * 4
    if c["context"] in ("gather", "host", "layers", "rope"):
        nbytes += rows * n_ret * nf * kv               # the gathered copy is a result
    elif c["context"] == "inplace_rope":
        nbytes += rows * n_ret * nf * kv / 2           # the re-positioned keys are
    n = n_ret * nf
    return {"bytes": nbytes, "flops": per_pair * rows * (nt * n + nt * (nt + 1) // 2) + 4.0 * rows * F * dim}


def tolerance(case):
    # About four times what the path was seen to lie from the same sums in 64 bits.  bf16: outputs and
    # probabilities keep 8 bits of mantissa (seen: 1.3e-3 of the norm, one unit in the last place at
    # most).  fp32: 3.5e-7 of the norm on the tiny stream; longer sums get some room.  Selections may
    # trade places only where two scores tie to the last bits.
    if case["dtype"] == "bf16":
        return {"rel": 5e-3, "max": 0.03, "differ": 2e-3}
    return {"rel": 4e-6, "max": 4e-5, "differ": 2e-3}
