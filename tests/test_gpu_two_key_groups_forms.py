"""The forms of the two-group 128-row kernel beside those of test_gpu_two_key_groups.py: one row block per question (streamed
tiles), values read in place beside re-positioned keys in a dense buffer, and infinities and NaN through both of its merges
(the two groups in LDS, the row block's last arriver), against the oracle."""
import numpy as np
import pytest
import torch

from oracle import rekv_oracle as O
from paper_2503_00540_amd.rekv import Rekv
from test_attention_plan import plan
from test_gpu_two_key_groups import QUESTIONS, key_groups
from test_gpu_wave_attention import agrees, bf16, dev

gpu = pytest.mark.gpu
DEV = "cuda:0"

ONE_BLOCK = [   # heads, new tokens, retrieved tokens, text, questions, several workgroups per row block
    (8, 2, 128, 10, 1500, 10, 16, True),          # 40 rows: two row waves of four
    (64, 8, 128, 10, 700, 33, 16, True),
    (14, 2, 64, 16, 2500, 16, 24, True),
    (16, 8, 64, 40, 1500, 45, 24, False),
    (64, 8, 128, 16, 700, 16, 24, False),         # 128 rows
]


@pytest.mark.parametrize("hq,hkv,d,n_new,n_ret,n_text,nq,several", ONE_BLOCK)
def test_these_take_two_groups_and_one_block(hq, hkv, d, n_new, n_ret, n_text, nq, several):
    assert key_groups(hq, hkv, d, n_new, n_ret, n_text, nq) == 2
    _, splits, row_blocks, *_ = plan(hq, hkv, d, n_new, n_ret, n_text, nq)
    assert row_blocks == 1 and (splits > 1) == several


@gpu
@pytest.mark.parametrize("hq,hkv,d,n_new,n_ret,n_text,nq,several", ONE_BLOCK)
def test_one_row_block_matches_oracle(hq, hkv, d, n_new, n_ret, n_text, nq, several):
    print(hq, hkv, d, n_new, n_ret, n_text, nq, flush=True)
    rng = np.random.default_rng(n_ret + hq)
    r = Rekv(hq, hkv, d, 1)
    q, kr, vr = bf16(rng, nq, n_new, hq, d), bf16(rng, nq, n_ret, hkv, d), bf16(rng, nq, n_ret, hkv, d)
    kt, vt = bf16(rng, nq, n_text, hkv, d), bf16(rng, nq, n_text, hkv, d)
    args = [dev(x) for x in (q, kr, vr, kt, vt)]
    valid = ([n_ret, 0, 1, 31, 33, n_ret // 2, n_ret - 1, 64] * 3)[:nq]
    n_sel = torch.tensor(valid, dtype=torch.int32, device=DEV)
    outs = [r.decode_attention(*args, n_text, n_sel=n_sel, no_alloc=i == 1) for i in range(3)]
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    got = outs[0].float().cpu().numpy()
    for i, n in enumerate(valid):
        assert agrees(got[i], O.decode_attention(q[i], kr[i, :n], vr[i, :n], kt[i], vt[i])), (i, n)


@gpu
@pytest.mark.parametrize("hq,hkv,d,n_new,n_ret,n_text,nq,several", [QUESTIONS[0], QUESTIONS[2], QUESTIONS[3]])
def test_values_in_place_beside_dense_keys_match_oracle(hq, hkv, d, n_new, n_ret, n_text, nq, several):
    n_f = 100
    frames, arena = n_ret // n_f, n_ret // n_f + 9
    assert key_groups(hq, hkv, d, n_new, frames * n_f, n_text, nq, in_place=True) == 2
    rng = np.random.default_rng(n_ret)
    r = Rekv(hq, hkv, d, n_f)
    k, v = bf16(rng, arena * n_f, hkv, d), bf16(rng, arena * n_f, hkv, d)
    q, kt, vt = bf16(rng, nq, n_new, hq, d), bf16(rng, nq, n_text, hkv, d), bf16(rng, nq, n_text, hkv, d)
    idx = np.stack([np.sort(rng.choice(arena, frames, replace=False)) for _ in range(nq)]).astype(np.int32)
    valid = ([frames, 1, 0, frames - 1, 2, frames] * 2)[:nq]
    n_sel = torch.tensor(valid, dtype=torch.int32, device=DEV)
    outs = [r.attention_indexed_rope(dev(q), dev(k), dev(v), torch.from_numpy(idx).to(DEV), dev(kt), dev(vt), n_text, n_sel=n_sel, pos_offset=7)
            for _ in range(3)]
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][0], outs[2][0])
    k_pos = outs[0][1].float().cpu().numpy()                 # (bit for bit the gather's: test_gpu_chain.py)
    for i, n in enumerate(valid):
        rv = O.gather_kv(k, v, idx[i, :n], n_f)[1] if n else v[:0]
        ref = O.decode_attention(q[i], k_pos[i, :n * n_f], rv, kt[i], vt[i])
        assert agrees(outs[0][0][i].float().cpu().numpy(), ref), (i, n)


@gpu
@pytest.mark.parametrize("case", [QUESTIONS[0], QUESTIONS[2], QUESTIONS[3], ONE_BLOCK[1], ONE_BLOCK[3]])
@pytest.mark.parametrize("where", ["q", "k", "v"])
def test_infinities_and_nan_stay_with_the_rows_that_see_them(case, where):
    """One question's input holds an infinity, another's a NaN, in keys (or values) of either half of the keys: what they make
    of their rows is what the oracle makes of them, and the other questions' results are bit for bit as without them."""
    hq, hkv, d, n_new, n_ret, n_text, nq, _ = case
    print(case, where, flush=True)
    rng = np.random.default_rng(5)
    r = Rekv(hq, hkv, d, 1)
    x = {"q": bf16(rng, nq, n_new, hq, d), "k": bf16(rng, nq, n_ret, hkv, d), "v": bf16(rng, nq, n_ret, hkv, d)}
    kt, vt = bf16(rng, nq, n_text, hkv, d), bf16(rng, nq, n_text, hkv, d)
    run = lambda: r.decode_attention(dev(x["q"]), dev(x["k"]), dev(x["v"]), dev(kt), dev(vt), n_text).float().cpu().numpy()
    clean = run()
    x[where] = x[where].copy()
    n = x[where].shape[1]
    x[where][1, 2, 0, 5] = np.inf
    x[where][2, n - 1, -1, 9] = np.nan
    x[where][3, n // 2, 0, 3] = -np.inf
    got = run()
    for i in range(nq):
        if i not in (1, 2, 3):
            assert np.array_equal(got[i], clean[i]), i
            continue
        with np.errstate(invalid="ignore"):
            ref = O.decode_attention(x["q"][i], x["k"][i], x["v"][i], kt[i], vt[i])
        assert np.array_equal(np.isnan(got[i]), np.isnan(ref)), i
        assert np.array_equal(np.isinf(got[i]), np.isinf(ref)) and (np.sign(got[i]) == np.sign(ref))[np.isinf(ref)].all(), i
        finite = np.isfinite(ref)
        assert 0 < finite.sum() < finite.size and agrees(got[i][finite], ref[finite]), i
