"""bf16 attention launches that are split over the keys inside a workgroup (few query rows): the sizes
where that split can go wrong - row counts around a block of 32 and 64 rows, tile counts around the
number of key runs, launches whose row blocks are shared by several workgroups - against the oracle.
Every call runs three times: the arrival counters must be back at zero after each launch."""
import numpy as np
import pytest
import torch

from oracle import rekv_oracle as O
from paper_2503_00540_amd import workloads as W
from paper_2503_00540_amd.rekv import Rekv
from test_attention_plan import plan

gpu = pytest.mark.gpu
DEV = "cuda:0"


def agrees(got, ref):
    """Against the oracle, relative to the result: over thousands of keys outputs are averages of a hundredth.  The output's
    rounding (2^-9 of a value, 1.1e-3 of the norm) and the probabilities' (as much again, they average like the values) make 1.6 to
    2.5e-3 of the norm; one element differs by some of these."""
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    rms = np.sqrt((ref ** 2).mean())
    diff = np.abs(got - ref)
    return np.sqrt((diff ** 2).mean()) < 5e-3 * rms and (diff < 0.03 * np.maximum(rms, np.abs(ref))).all()


def bf16(rng, *shape):
    return W.round_to_bf16(rng.standard_normal(shape))


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(torch.bfloat16).to(DEV)


def test_the_bound_sees_a_lost_key_range():
    """What a merge that drops one of 25 workgroups' key ranges, or one tile of 32 keys, would give is refused."""
    rng = np.random.default_rng(1)
    hq, hkv, d, n = 4, 1, 128, 12641
    q, k, v = bf16(rng, 1, hq, d), bf16(rng, n, hkv, d), bf16(rng, n, hkv, d)
    own = k[-1:], v[-1:]
    ref = O.decode_attention(q, k[:-1], v[:-1], *own)
    assert agrees(W.round_to_bf16(ref), ref)
    for lost in (n // 25, 32):
        keep = np.r_[0:5000, 5000 + lost:n - 1]
        assert not agrees(O.decode_attention(q, k[keep], v[keep], *own), ref)


@gpu
@pytest.mark.parametrize("hq,hkv,d,n_new,n_ret,n_text,row_waves", [
    (1, 1, 128, 1, 0, 1, 0),            # one row, one key: the 128-row kernel
    (7, 1, 128, 1, 31, 5, 0),
    (8, 1, 128, 4, 224, 32, 1),         # exactly 32 rows, exactly 8 tiles
    (1, 1, 128, 1, 150, 8, 1),          # fewer tiles than key runs
    (3, 1, 64, 11, 225, 40, 1),         # 33 rows: a block of one row; a tile of one key
    (16, 2, 64, 4, 4000, 9, 0),
    (28, 4, 128, 9, 1500, 20, 1),       # 63 rows
    (28, 4, 128, 32, 3136, 32, 1),      # a question of the 7B-class shapes
    (8, 8, 128, 65, 700, 65, 1),        # one head per group, 65 rows, causal part over three tiles
    (28, 4, 128, 1, 12544, 97, 1),      # a decode step split over many workgroups
])
def test_few_rows_match_oracle(hq, hkv, d, n_new, n_ret, n_text, row_waves):
    rng = np.random.default_rng(hq * 1000 + n_new)
    r = Rekv(hq, hkv, d, 1)
    for nq in (1, 3):
        assert plan(hq, hkv, d, n_new, n_ret, n_text, nq)[0] == row_waves
        q, kr, vr = bf16(rng, nq, n_new, hq, d), bf16(rng, nq, n_ret, hkv, d), bf16(rng, nq, n_ret, hkv, d)
        kt, vt = bf16(rng, nq, n_text, hkv, d), bf16(rng, nq, n_text, hkv, d)
        args = [dev(x) for x in (q, kr, vr, kt, vt)]
        outs = [r.decode_attention(*args, n_text, no_alloc=bool(i % 2)) for i in range(3)]
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
        got = outs[0].float().cpu().numpy()
        for i in range(nq):
            assert agrees(got[i], O.decode_attention(q[i], kr[i], vr[i], kt[i], vt[i]))


# every way through the kernel: row waves, split or not, and what the last arriver's threads do with its row block's chunks
PATHS = [
    (8, 8, 64, 65, 300, 72, 2, (1, False)),
    (2, 2, 64, 3, 6000, 3, 2, (1, True)),            # thread groups share the splits
    (3, 1, 64, 17, 3136, 24, 1, (1, True)),          # a chunk per thread
    (56, 8, 64, 48, 300, 48, 3, (2, False)),
    (24, 8, 64, 33, 3136, 33, 3, (2, True)),         # several chunks per thread
    (56, 8, 64, 48, 3136, 55, 1, (2, True)),         # and a last block of 16 rows, by thread groups
    (1, 1, 128, 1, 300, 8, 1, (1, False)),
    (2, 2, 128, 1, 6000, 1, 2, (1, True)),
    (5, 1, 128, 9, 1500, 16, 1, (1, True)),
    (3, 1, 128, 17, 1500, 24, 1, (1, True)),
    (40, 8, 128, 65, 300, 72, 3, (2, False)),
    (28, 4, 128, 33, 3136, 40, 3, (2, True)),
    (28, 4, 128, 65, 3136, 65, 2, (2, True)),        # a last block of seven rows
]


@gpu
@pytest.mark.parametrize("hq,hkv,d,n_new,n_ret,n_text,nq,want", PATHS)
def test_every_path_matches_oracle(hq, hkv, d, n_new, n_ret, n_text, nq, want):
    """All retrieved tokens valid, then as few as none: key ranges without a tile take part in the merge."""
    print(hq, hkv, d, n_new, n_ret, n_text, nq, flush=True)
    chosen = plan(hq, hkv, d, n_new, n_ret, n_text, nq)
    assert (chosen[0], chosen[1] > 1) == want
    rng = np.random.default_rng(n_ret + hq)
    r = Rekv(hq, hkv, d, 1)
    q, kr, vr = bf16(rng, nq, n_new, hq, d), bf16(rng, nq, n_ret, hkv, d), bf16(rng, nq, n_ret, hkv, d)
    kt, vt = bf16(rng, nq, n_text, hkv, d), bf16(rng, nq, n_text, hkv, d)
    args = [dev(x) for x in (q, kr, vr, kt, vt)]
    for valid in ([n_ret] * nq, [1, n_ret // 3, 0][:nq], [0, 33, n_ret - 1][:nq]):
        n_sel = torch.tensor(valid, dtype=torch.int32, device=DEV)
        outs = [r.decode_attention(*args, n_text, n_sel=n_sel, no_alloc=bool(i)) for i in range(2)]
        assert torch.equal(outs[0], outs[1])
        got = outs[0].float().cpu().numpy()
        for i, n in enumerate(valid):
            assert agrees(got[i], O.decode_attention(q[i], kr[i, :n], vr[i, :n], kt[i], vt[i])), (i, n)


@gpu
@pytest.mark.parametrize("n_ret", [975_343, 1_045_000])
def test_the_longest_context_matches_oracle(n_ret):
    """One row over a million keys: the most splits the last arriver's LDS has room for."""
    wave, splits, *_ = plan(1, 1, 64, 1, n_ret, 1)
    assert wave == 1 and splits > 200
    g = torch.Generator().manual_seed(n_ret)
    q, kr, vr, kt, vt = [torch.randn((1, n, 1, 64), generator=g).bfloat16() for n in (1, n_ret, n_ret, 1, 1)]
    r = Rekv(1, 1, 64, 1)
    outs = [r.decode_attention(*(x.to(DEV) for x in (q, kr, vr, kt, vt)), 1, no_alloc=bool(i)) for i in range(2)]
    assert torch.equal(outs[0], outs[1])
    ref = O.decode_attention(*(x[0].double().numpy() for x in (q, kr, vr, kt, vt)))
    assert agrees(outs[0][0].float().cpu().numpy(), ref)


@gpu
@pytest.mark.parametrize("hq,hkv,d,n_new,frames,n_f,nq,want", [
    (3, 1, 64, 17, 64, 49, 1, (1, True)),
    (24, 8, 64, 33, 64, 49, 3, (2, True)),
    (2, 2, 128, 1, 60, 101, 2, (1, True)),
    (28, 4, 128, 65, 16, 196, 2, (2, True)),
])
def test_split_launches_through_a_frame_list_match_oracle(hq, hkv, d, n_new, frames, n_f, nq, want):
    n_text, arena = n_new + 3, frames + 9
    chosen = plan(hq, hkv, d, n_new, frames * n_f, n_text, nq, in_place=True)
    assert (chosen[0], chosen[1] > 1) == want
    rng = np.random.default_rng(frames)
    r = Rekv(hq, hkv, d, n_f)
    k, v = bf16(rng, arena * n_f, hkv, d), bf16(rng, arena * n_f, hkv, d)
    q, kt, vt = bf16(rng, nq, n_new, hq, d), bf16(rng, nq, n_text, hkv, d), bf16(rng, nq, n_text, hkv, d)
    idx = np.stack([np.sort(rng.choice(arena, frames, replace=False)) for _ in range(nq)]).astype(np.int32)
    for valid in ([frames] * nq, [1, frames - 1, 0][:nq]):
        n_sel = torch.tensor(valid, dtype=torch.int32, device=DEV)
        outs = [r.attention_indexed(dev(q), dev(k), dev(v), torch.from_numpy(idx).to(DEV), frames, dev(kt), dev(vt), n_text, n_sel=n_sel)
                for _ in range(2)]
        assert torch.equal(outs[0], outs[1])
        for i, n in enumerate(valid):
            rk, rv = O.gather_kv(k, v, idx[i, :n], n_f) if n else (k[:0], v[:0])
            assert agrees(outs[0][i].float().cpu().numpy(), O.decode_attention(q[i], rk, rv, kt[i], vt[i])), (i, n)


@gpu
@pytest.mark.parametrize("hq,hkv,d,l_x,n_chunks,l_l,first,want", [
    (28, 4, 128, 196, 1, 16 * 196, 16 * 196, (1, False)),    # a live frame, window full
    (14, 2, 64, 196, 1, 16 * 196, 16 * 196, (1, True)),
    (28, 4, 128, 37, 2, 100, 60, (1, False)),                # window not full, ragged everything
    (64, 8, 128, 144, 1, 500, 2000, (2, False)),             # 64-row blocks shared by two waves
    (28, 4, 128, 144, 1, 3136, 3200, (2, True)),             # and by several workgroups
    (14, 2, 64, 588, 1, 1960, 2000, (2, True)),
    (4, 4, 64, 33, 1, 0, 0, (0, False)),                     # no window: the 128-row kernel
])
def test_live_chunks_match_oracle(hq, hkv, d, l_x, n_chunks, l_l, first, want):
    rng = np.random.default_rng(l_x + hq)
    r = Rekv(hq, hkv, d, 1)
    chosen = plan(hq, hkv, d, l_x, l_l, l_x, n_chunks, True, first)
    assert (chosen[0], chosen[1] > 1) == want
    n = first + n_chunks * l_x
    q, k, v = bf16(rng, n_chunks * l_x, hq, d), bf16(rng, n, hkv, d), bf16(rng, n, hkv, d)
    dq, dk, dv = dev(q), dev(k), dev(v)
    outs = [r.encode_chunk(dq, dk, dv, first, l_x, n_chunks, l_l) for _ in range(3)]
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    ref = O.encode_chunks(q, k, v, first, l_x, n_chunks, l_l)
    assert agrees(outs[0].float().cpu().numpy(), ref)


@gpu
def test_captured_no_alloc_call_outlives_its_context():
    """The allocation-free call keeps its scratch and its arrival counters when the context is gone."""
    g = torch.Generator().manual_seed(2)
    q, kr, vr, kt, vt = [torch.randn((1, n, h, 128), generator=g).bfloat16().cuda()
                         for n, h in ((1, 28), (12544, 4), (12544, 4), (97, 4), (97, 4))]
    assert plan(28, 4, 128, 1, 12544, 97)[0] == 1 and plan(28, 4, 128, 1, 12544, 97)[1] > 1
    r = Rekv(28, 4, 128, 196, "bf16")
    want = r.decode_attention(q, kr, vr, kt, vt, 97)
    out = torch.empty_like(q)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        r.decode_attention(q, kr, vr, kt, vt, 97, out=out, no_alloc=True)
    torch.cuda.synchronize()
    r.close()
    other = Rekv(28, 4, 128, 196, "bf16")
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(other.decode_attention(q, kr, vr, kt, vt, 97), want)


@gpu
def test_captured_no_alloc_call_beside_its_contexts_other_calls():
    """A replayed allocation-free call on one stream, split attention and retrieval of the same context on another:
    they have no counters and no scratch in common."""
    g = torch.Generator().manual_seed(5)
    q, kr, vr, kt, vt = [torch.randn((1, n, h, 128), generator=g).bfloat16().to(DEV)
                         for n, h in ((1, 28), (12544, 4), (12544, 4), (97, 4), (97, 4))]
    qq, qk, qv = [torch.randn((1, 32, h, 128), generator=g).bfloat16().to(DEV) for h in (28, 4, 4)]
    table = torch.randn((200, 512), generator=g).to(DEV)
    short = kr[:, :3136].contiguous(), vr[:, :3136].contiguous()
    for n_new, n_ret, n_text in ((1, 12544, 97), (32, 3136, 32)):
        chosen = plan(28, 4, 128, n_new, n_ret, n_text)
        assert chosen[0] == 1 and chosen[1] > 1
    r = Rekv(28, 4, 128, 196)
    want = r.decode_attention(q, kr, vr, kt, vt, 97)
    want_qa, want_idx = r.qa_attention(qq, *short, qk, qv), r.retrieve_topk(table, 200, qq, 16)[0]
    out = torch.empty_like(q)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        for _ in range(20):
            r.decode_attention(q, kr, vr, kt, vt, 97, out=out, no_alloc=True)
    torch.cuda.synchronize()
    for _ in range(5):
        out.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            graph.replay()
        got = [(r.qa_attention(qq, *short, qk, qv), r.retrieve_topk(table, 200, qq, 16)[0]) for _ in range(10)]
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert all(torch.equal(a, want_qa) and torch.equal(i, want_idx) for a, i in got)


@gpu
def test_more_contexts_than_static_counter_slots():
    """70 contexts at once, each on a stream of its own; destroyed with their work still queued, and 70 more."""
    g = torch.Generator().manual_seed(6)
    q, kr, vr, kt, vt = [torch.randn((1, n, h, 128), generator=g).bfloat16().to(DEV)
                         for n, h in ((32, 28), (3136, 4), (3136, 4), (32, 4), (32, 4))]
    want = Rekv(28, 4, 128, 196).qa_attention(q, kr, vr, kt, vt)
    streams = [torch.cuda.Stream() for _ in range(8)]
    torch.cuda.synchronize()
    for _ in range(2):
        got = []
        contexts = [Rekv(28, 4, 128, 196) for _ in range(70)]
        for i, r in enumerate(contexts):
            with torch.cuda.stream(streams[i % 8]):
                got += [r.qa_attention(q, kr, vr, kt, vt) for _ in range(2)]
        for r in contexts:
            r.close()
        torch.cuda.synchronize()
        assert all(torch.equal(x, want) for x in got)


@gpu
def test_calls_captured_after_an_unsplit_launch_need_no_allocation():
    """A live frame that one workgroup per row block serves leaves the workspace that splitting it would have left, so
    that a question's retrieval and attention can be captured before they ever ran."""
    g = torch.Generator().manual_seed(7)
    mk = lambda *s: torch.randn(s, generator=g).bfloat16().to(DEV)
    r, other = Rekv(28, 4, 128, 196), Rekv(28, 4, 128, 196)
    assert plan(28, 4, 128, 196, 16 * 196, 196, encode=True)[1] == 1
    k, v = mk(17 * 196, 4, 128), mk(17 * 196, 4, 128)
    r.encode_chunk(mk(196, 28, 128), k, v, 16 * 196, 196, 1, 16 * 196)
    q, kr, vr, ks, vs = mk(1, 32, 28, 128), mk(1, 3136, 4, 128), mk(1, 3136, 4, 128), mk(1, 32, 4, 128), mk(1, 32, 4, 128)
    table = torch.randn((900, 512), generator=g).to(DEV)
    assert plan(28, 4, 128, 32, 3136, 32)[1] > 1
    want = other.qa_attention(q, kr, vr, ks, vs), other.retrieve_topk(table, 900, q, 16)[0]
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        got = r.qa_attention(q, kr, vr, ks, vs), r.retrieve_topk(table, 900, q, 16)[0]
    torch.cuda.synchronize()
    for _ in range(3):
        for x in got:
            x.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
