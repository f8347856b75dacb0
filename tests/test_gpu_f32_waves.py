"""fp32 attention around the key counts where its launch takes one, four or eight wavefronts per row block (one step of 32
keys, 16 at head_dim 128; four steps), also where an item has fewer keys than the launch was sized for - against the oracle."""
import numpy as np
import pytest
import torch

from oracle import rekv_oracle as O
from paper_2503_00540_amd.rekv import Rekv
from test_gpu_f32_attention import DEV, TOL, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("steps", [1, 4])
@pytest.mark.parametrize("over", [-1, 0, 1])
def test_questions(d, steps, over):
    hq, hkv, n_new = 6, 2, 5
    n = steps * (32 if d == 64 else 16) + over - n_new           # retrieved keys
    rng = np.random.default_rng(n)
    r = Rekv(hq, hkv, d, 1, "f32")
    g = lambda *shape: rng.standard_normal(shape).astype(np.float32)
    q, kr, vr, kt, vt = g(2, n_new, hq, d), g(2, n, hkv, d), g(2, n, hkv, d), g(2, n_new, hkv, d), g(2, n_new, hkv, d)
    valid = [n, n // 2]
    n_sel = torch.tensor(valid, dtype=torch.int32, device=DEV)
    got = r.decode_attention(dev(q), dev(kr), dev(vr), dev(kt), dev(vt), n_new, n_sel=n_sel).cpu().numpy()
    for i, m in enumerate(valid):
        assert np.abs(got[i] - O.decode_attention(q[i], kr[i, :m], vr[i, :m], kt[i], vt[i])).max() < TOL


@pytest.mark.parametrize("l_x,n_chunks,l_l,first", [(16, 4, 64, 0), (32, 3, 0, 5), (16, 3, 16, 0), (33, 2, 95, 40), (20, 3, 1000, 10)])
def test_chunks(l_x, n_chunks, l_l, first):
    rng = np.random.default_rng(l_x)
    n = first + n_chunks * l_x
    q, k, v = (rng.standard_normal((m, h, 64)).astype(np.float32) for m, h in ((n_chunks * l_x, 4), (n, 1), (n, 1)))
    got = Rekv(4, 1, 64, 1, "f32").encode_chunk(dev(q), dev(k), dev(v), first, l_x, n_chunks, l_l).cpu().numpy()
    assert np.abs(got - O.encode_chunks(q, k, v, first, l_x, n_chunks, l_l)).max() < TOL
