"""fp32 attention on the matrix cores (head_dim 64 and 128) where its tiling can go wrong: row counts
around the 16-row block, key counts around a step of 32 (16 at head_dim 128) keys, one, four and eight
wavefronts per row block, keys through a frame index list - against the oracle."""
import numpy as np
import pytest
import torch

from oracle import rekv_oracle as O
from paper_2503_00540_amd.rekv import Rekv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# scores are sums of up to 128 products (relative error 128 * 2^-24 = 8e-6 of values below 10, entering the
# probabilities as an absolute error); outputs are averages of values below 5
TOL = 1e-4


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(DEV)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv,n_new,n_ret,n_text,nq", [
    (1, 1, 1, 0, 1, 1),              # one row, one key
    (5, 1, 3, 16, 3, 2),             # 15 rows
    (8, 2, 4, 31, 20, 1),            # 16 rows, 31 + 20 keys
    (17, 1, 1, 33, 1, 3),            # 17 rows
    (4, 2, 40, 500, 45, 2),          # causal part over several steps
    (4, 4, 64, 60, 64, 70),          # 1,120 row blocks: four wavefronts each
])
def test_matches_oracle(d, hq, hkv, n_new, n_ret, n_text, nq):
    rng = np.random.default_rng(hq * 100 + n_new)
    r = Rekv(hq, hkv, d, 1, "f32")
    g = lambda *shape: rng.standard_normal(shape).astype(np.float32)
    q, kr, vr = g(nq, n_new, hq, d), g(nq, n_ret, hkv, d), g(nq, n_ret, hkv, d)
    kt, vt = g(nq, n_text, hkv, d), g(nq, n_text, hkv, d)
    got = r.decode_attention(dev(q), dev(kr), dev(vr), dev(kt), dev(vt), n_text).cpu().numpy()
    for i in range(0, nq, 7):
        ref = O.decode_attention(q[i], kr[i], vr[i], kt[i], vt[i])
        assert np.abs(got[i] - ref).max() < TOL


def test_many_row_blocks_match_oracle():
    """4,160 row blocks: one wavefront each."""
    hq, hkv, d, l_x, n_chunks, l_l = 7, 1, 64, 37, 256, 75
    rng = np.random.default_rng(3)
    n = n_chunks * l_x
    q, k, v = (rng.standard_normal((n, h, d)).astype(np.float32) for h in (hq, hkv, hkv))
    got = Rekv(hq, hkv, d, 1, "f32").encode_chunk(dev(q), dev(k), dev(v), 0, l_x, n_chunks, l_l).cpu().numpy()
    for c in (0, 1, 2, 100, 255):
        sl = slice(c * l_x, (c + 1) * l_x)
        ref = O.encode_chunks(q[sl], k, v, c * l_x, l_x, 1, l_l)
        assert np.abs(got[sl] - ref).max() < TOL


@pytest.mark.parametrize("n_f,frames", [(7, 9), (16, 4), (33, 2)])
def test_indexed_keys_match_oracle(n_f, frames):
    hq, hkv, d, n_new, n_text = 6, 2, 64, 5, 9
    rng = np.random.default_rng(n_f)
    r = Rekv(hq, hkv, d, n_f, "f32")
    g = lambda *shape: rng.standard_normal(shape).astype(np.float32)
    k, v = g(40 * n_f, hkv, d), g(40 * n_f, hkv, d)
    q, kt, vt = g(2, n_new, hq, d), g(2, n_text, hkv, d), g(2, n_text, hkv, d)
    idx = np.stack([np.sort(rng.choice(40, frames, replace=False)) for _ in range(2)]).astype(np.int32)
    got = r.attention_indexed(dev(q), dev(k), dev(v), torch.from_numpy(idx).to(DEV), frames, dev(kt), dev(vt), n_text).cpu().numpy()
    for i in range(2):
        rk, rv = O.gather_kv(k, v, idx[i], n_f)
        assert np.abs(got[i] - O.decode_attention(q[i], rk, rv, kt[i], vt[i])).max() < TOL


@pytest.mark.parametrize("d", [64, 128, 32])          # 32: the kernel on the vector ALU
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("n_ret,n_text,n_new,hq,nq", [(0, 9, 9, 2, 1), (37, 50, 20, 3, 1), (200, 33, 33, 8, 40), (16, 40, 1, 16, 2)])
def test_values_no_row_sees_stay_out(d, bad, n_ret, n_text, n_new, hq, nq):
    """An infinity or NaN in a text token's value reaches exactly the rows that see the token, whatever shares a tile or a
    row block with them; in the last visible key, which fills up ragged tiles, it stays what it is."""
    rng = np.random.default_rng(n_text)
    r = Rekv(hq, 1, d, 1, "f32")
    g = lambda *shape: rng.standard_normal(shape).astype(np.float32)
    q, kr, vr, kt, vt = g(nq, n_new, hq, d), g(nq, n_ret, 1, d), g(nq, n_ret, 1, d), g(nq, n_text, 1, d), g(nq, n_text, 1, d)
    for at in sorted({n_text - n_new, n_text - n_new // 2 - 1, n_text - 1}):
        broken = vt.copy()
        broken[:, at, 0, ::3] = bad
        got = r.decode_attention(dev(q), dev(kr), dev(vr), dev(kt), dev(broken), n_text).cpu().numpy()
        seen = np.arange(n_text - n_new, n_text) >= at               # rows that see token `at`
        for i in range(0, nq, 13):
            ref = O.decode_attention(q[i], kr[i], vr[i], kt[i], vt[i])
            assert np.abs(got[i][~seen] - ref[~seen]).max(initial=0) < TOL
            assert np.abs(got[i][seen][..., 1::3] - ref[seen][..., 1::3]).max(initial=0) < TOL
            hit = got[i][seen][..., ::3]
            assert np.isnan(hit).all() if np.isnan(bad) else (hit == bad).all()
