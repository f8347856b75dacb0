"""128-row attention launches whose workgroups divide the keys between two groups of four wavefronts: runs of unequal
length and without a tile, last blocks with one or all of their row waves, one and several workgroups per row
block, windows that are not full, against the oracle.  Every call runs three times: the arrival counters
must be back at zero after each launch, and the result must not depend on which workgroup came last."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import rekv_oracle as O
from paper_2503_00540_amd import rekv
from paper_2503_00540_amd.rekv import Rekv
from test_attention_plan import plan
from test_gpu_wave_attention import agrees, bf16, dev

gpu = pytest.mark.gpu
DEV = "cuda:0"


def key_groups(hq, hkv, d, len_q, len_a, len_b, items=1, encode=False, first=1 << 40, in_place=False):
    f = rekv.lib().rekv_internal_attention_key_groups
    f.restype = ctypes.c_int32
    f.argtypes = [ctypes.c_int32] * 4 + [ctypes.c_int64] + [ctypes.c_int32] * 5
    return f(hq, hkv, d, int(encode), first, items, len_q, len_a, len_b, int(in_place))


QUESTIONS = [   # heads, new tokens, retrieved tokens, text, questions, several workgroups per row block
    (64, 8, 128, 33, 2500, 33, 4, True),
    (64, 8, 128, 17, 5000, 30, 8, True),          # a last block of one row wave
    (64, 8, 128, 48, 1100, 48, 8, False),
    (14, 2, 64, 130, 3200, 130, 6, True),
    (8, 2, 128, 129, 2400, 140, 9, True),
]
CHUNKS = [      # heads, chunk, chunks, window, first token, several
    (28, 4, 128, 196, 1, 40 * 196, 41 * 196, True),
    (28, 4, 128, 784, 1, 900, 1000, False),
    (64, 8, 128, 288, 1, 2304, 2400, False),
    (8, 2, 128, 300, 4, 4000, 350, True),         # the first chunks' windows are not full: runs without a tile
    (16, 8, 64, 392, 1, 60 * 196, 60 * 196, True),
]


@pytest.mark.parametrize("hq,hkv,d,n_new,n_ret,n_text,nq,several", QUESTIONS)
def test_these_questions_take_two_groups(hq, hkv, d, n_new, n_ret, n_text, nq, several):
    for in_place in (False, True):
        assert key_groups(hq, hkv, d, n_new, n_ret, n_text, nq, in_place=in_place) == 2
        assert (plan(hq, hkv, d, n_new, n_ret, n_text, nq, in_place=in_place)[1] > 1) == several


@pytest.mark.parametrize("hq,hkv,d,l_x,n_chunks,l_l,first,several", CHUNKS)
def test_these_chunks_take_two_groups(hq, hkv, d, l_x, n_chunks, l_l, first, several):
    assert key_groups(hq, hkv, d, l_x, l_l, l_x, n_chunks, True, first) == 2
    assert (plan(hq, hkv, d, l_x, l_l, l_x, n_chunks, True, first)[1] > 1) == several


@gpu
@pytest.mark.parametrize("hq,hkv,d,n_new,n_ret,n_text,nq,several", QUESTIONS)
def test_questions_match_oracle(hq, hkv, d, n_new, n_ret, n_text, nq, several):
    print(hq, hkv, d, n_new, n_ret, n_text, nq, flush=True)
    rng = np.random.default_rng(n_ret)
    r = Rekv(hq, hkv, d, 1)
    q, kr, vr = bf16(rng, nq, n_new, hq, d), bf16(rng, nq, n_ret, hkv, d), bf16(rng, nq, n_ret, hkv, d)
    kt, vt = bf16(rng, nq, n_text, hkv, d), bf16(rng, nq, n_text, hkv, d)
    args = [dev(x) for x in (q, kr, vr, kt, vt)]
    for valid in ([n_ret] * nq, ([0, 1, 31, 33, n_ret // 2, n_ret - 1, 0, 64, 700])[:nq]):
        n_sel = torch.tensor(valid, dtype=torch.int32, device=DEV)
        outs = [r.decode_attention(*args, n_text, n_sel=n_sel, no_alloc=i == 1) for i in range(3)]
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
        got = outs[0].float().cpu().numpy()
        for i, n in enumerate(valid):
            assert agrees(got[i], O.decode_attention(q[i], kr[i, :n], vr[i, :n], kt[i], vt[i])), (i, n)


@gpu
@pytest.mark.parametrize("hq,hkv,d,n_new,n_ret,n_text,nq,several", [QUESTIONS[0], QUESTIONS[3]])
def test_questions_read_in_place_match_oracle(hq, hkv, d, n_new, n_ret, n_text, nq, several):
    n_f = 100
    frames, arena = n_ret // n_f, n_ret // n_f + 9
    rng = np.random.default_rng(n_ret)
    r = Rekv(hq, hkv, d, n_f)
    k, v = bf16(rng, arena * n_f, hkv, d), bf16(rng, arena * n_f, hkv, d)
    q, kt, vt = bf16(rng, nq, n_new, hq, d), bf16(rng, nq, n_text, hkv, d), bf16(rng, nq, n_text, hkv, d)
    idx = np.stack([np.sort(rng.choice(arena, frames, replace=False)) for _ in range(nq)]).astype(np.int32)
    valid = [frames, 1, 0, frames - 1, 2, frames][:nq]
    n_sel = torch.tensor(valid, dtype=torch.int32, device=DEV)
    outs = [r.attention_indexed(dev(q), dev(k), dev(v), torch.from_numpy(idx).to(DEV), frames, dev(kt), dev(vt), n_text, n_sel=n_sel)
            for _ in range(3)]
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    for i, n in enumerate(valid):
        rk, rv = O.gather_kv(k, v, idx[i, :n], n_f) if n else (k[:0], v[:0])
        assert agrees(outs[0][i].float().cpu().numpy(), O.decode_attention(q[i], rk, rv, kt[i], vt[i])), (i, n)


@gpu
@pytest.mark.parametrize("hq,hkv,d,l_x,n_chunks,l_l,first,several", CHUNKS)
def test_chunks_match_oracle(hq, hkv, d, l_x, n_chunks, l_l, first, several):
    print(hq, hkv, d, l_x, n_chunks, l_l, first, flush=True)
    rng = np.random.default_rng(l_x)
    r = Rekv(hq, hkv, d, 1)
    n = first + n_chunks * l_x
    q, k, v = bf16(rng, n_chunks * l_x, hq, d), bf16(rng, n, hkv, d), bf16(rng, n, hkv, d)
    dq, dk, dv = dev(q), dev(k), dev(v)
    outs = [r.encode_chunk(dq, dk, dv, first, l_x, n_chunks, l_l) for _ in range(3)]
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert agrees(outs[0].float().cpu().numpy(), O.encode_chunks(q, k, v, first, l_x, n_chunks, l_l))
