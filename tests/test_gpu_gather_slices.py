"""The block copy at the edges of its slices and grids: frames shorter than a 4 KB slice, exactly one, one 16-byte
chunk more, ragged; more blocks than a grid dimension holds; more slices than the host copy has workgroups.
Copies are exact; a rotation by position 0 changes nothing."""
import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPES = [                     # n_kv_heads, head_dim, tokens per frame, dtype; frame bytes
    (1, 4, 1, "f32"),          # 16
    (1, 64, 16, "f32"),        # 4,096: one slice
    (1, 4, 257, "f32"),        # 4,112: one chunk more
    (2, 64, 37, "bf16"),       # 9,472
    (4, 128, 196, "bf16"),     # 200,704: 49 slices
]


def arenas(shape, frames, seed):
    hkv, d, nf, dtype = shape
    g = torch.Generator().manual_seed(seed)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    return [torch.randn((frames * nf, hkv, d), generator=g).to(dt) for _ in range(2)]


def expected(x, idx, frames, nf):
    rows = x.view(frames, -1)
    bad = (idx < 0) | (idx >= frames)
    out = rows[idx.clamp(0, frames - 1).long().flatten()]
    out[bad.flatten()] = 0
    return out.view(idx.shape[0], idx.shape[1] * nf, *x.shape[1:])


@pytest.mark.parametrize("source", ["device", "host", "rope", "rope_host", "layers"])
@pytest.mark.parametrize("shape", SHAPES)
def test_block_copy(shape, source):
    from paper_2503_00540_amd.rekv import Rekv
    hkv, d, nf, dtype = shape
    if source.startswith("rope") and d % (8 if dtype == "f32" else 16):
        pytest.skip("head_dim too small to rotate")
    print(shape, source, flush=True)
    frames, nq, k = 23, 3, 7
    r = Rekv(hkv, hkv, d, nf, dtype)
    k_src, v_src = arenas(shape, frames, 5)
    idx = torch.randint(0, frames, (nq, k), generator=torch.Generator().manual_seed(6), dtype=torch.int32)
    idx[1, 5:] = -1
    idx[2, 6] = frames          # past the arena: zeros, like padding
    want = [expected(x, idx, frames, nf) for x in (k_src, v_src)]
    di = idx.to("cuda:0")
    on_host = source in ("host", "rope_host")
    src = [x.pin_memory() if on_host else x.to("cuda:0") for x in (k_src, v_src)]
    if source == "layers":
        got = r.gather_kv_layers([src[0]] * nq, [src[1]] * nq, di.view(nq, 1, k), n_src_frames=frames)
    elif source.startswith("rope"):
        got = r.gather_kv_rope(src[0], src[1], di, n_src_frames=frames, mode="static")
    else:
        got = r.gather_kv(src[0], src[1], di, n_src_frames=frames)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a.cpu().view(b.shape), b)


@pytest.mark.parametrize("on_host", [False, True])
def test_more_blocks_than_a_grid_dimension(on_host):
    from paper_2503_00540_amd.rekv import Rekv
    shape, frames, n = SHAPES[0], 50, 65535 + 70
    r = Rekv(1, 1, shape[1], shape[2], shape[3])
    k_src, v_src = arenas(shape, frames, 7)
    idx = torch.randint(0, frames, (1, n), generator=torch.Generator().manual_seed(8), dtype=torch.int32)
    src = [x.pin_memory() if on_host else x.to("cuda:0") for x in (k_src, v_src)]
    got = r.gather_kv(src[0], src[1], idx.to("cuda:0"), n_src_frames=frames)
    torch.cuda.synchronize()
    for a, x in zip(got, (k_src, v_src)):
        assert torch.equal(a.cpu(), expected(x, idx, frames, 1))
