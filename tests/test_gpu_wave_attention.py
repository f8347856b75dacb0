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

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# outputs are averages of N(0,1) values, below 4 in size: one bf16 rounding of the result (2^-9 * 4 = 8e-3)
# and the probabilities' roundings (2^-9 each, averaging out) stay below 2e-2
TOL = 2e-2


def bf16(rng, *shape):
    return W.round_to_bf16(rng.standard_normal(shape))


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(torch.bfloat16).to(DEV)


@pytest.mark.parametrize("hq,hkv,d,n_new,n_ret,n_text", [
    (1, 1, 128, 1, 0, 1),            # one row, one key
    (7, 1, 128, 1, 31, 5),           # fewer tiles than key runs
    (8, 1, 128, 4, 224, 32),         # exactly 32 rows, exactly 8 tiles
    (3, 1, 64, 11, 225, 40),         # 33 rows: a block of one row; a tile of one key
    (16, 2, 64, 4, 4000, 9),         # row blocks shared by workgroups
    (28, 4, 128, 9, 1500, 20),       # 63 rows
    (28, 4, 128, 32, 3136, 32),      # a question of the 7B-class shapes
    (8, 8, 128, 65, 700, 65),        # one head per group, 65 rows, causal part over three tiles
    (28, 4, 128, 1, 12544, 97),      # a decode step split over many workgroups
])
def test_few_rows_match_oracle(hq, hkv, d, n_new, n_ret, n_text):
    rng = np.random.default_rng(hq * 1000 + n_new)
    r = Rekv(hq, hkv, d, 1)
    for nq in (1, 3):
        q, kr, vr = bf16(rng, nq, n_new, hq, d), bf16(rng, nq, n_ret, hkv, d), bf16(rng, nq, n_ret, hkv, d)
        kt, vt = bf16(rng, nq, n_text, hkv, d), bf16(rng, nq, n_text, hkv, d)
        args = [dev(x) for x in (q, kr, vr, kt, vt)]
        outs = [r.decode_attention(*args, n_text, no_alloc=bool(i % 2)) for i in range(3)]
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
        got = outs[0].float().cpu().numpy()
        for i in range(nq):
            ref = O.decode_attention(q[i], kr[i], vr[i], kt[i], vt[i])
            assert np.abs(got[i] - ref).max() < TOL


@pytest.mark.parametrize("hq,hkv,d,l_x,n_chunks,l_l,first", [
    (28, 4, 128, 196, 1, 16 * 196, 16 * 196),    # a live frame, window full
    (14, 2, 64, 196, 1, 16 * 196, 16 * 196),
    (28, 4, 128, 37, 2, 100, 60),                # window not full, ragged everything
    (64, 8, 128, 144, 1, 500, 2000),             # 64-row blocks shared by two waves
    (4, 4, 64, 33, 1, 0, 0),                     # no window
])
def test_live_chunks_match_oracle(hq, hkv, d, l_x, n_chunks, l_l, first):
    rng = np.random.default_rng(l_x + hq)
    r = Rekv(hq, hkv, d, 1)
    n = first + n_chunks * l_x
    q, k, v = bf16(rng, n_chunks * l_x, hq, d), bf16(rng, n, hkv, d), bf16(rng, n, hkv, d)
    dq, dk, dv = dev(q), dev(k), dev(v)
    outs = [r.encode_chunk(dq, dk, dv, first, l_x, n_chunks, l_l) for _ in range(3)]
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    ref = O.encode_chunks(q, k, v, first, l_x, n_chunks, l_l)
    assert np.abs(outs[0].float().cpu().numpy() - ref).max() < TOL


def test_captured_no_alloc_call_outlives_its_context():
    """The allocation-free call keeps its scratch and its arrival counters when the context is gone."""
    import torch
    from paper_2503_00540_amd.rekv import Rekv
    g = torch.Generator().manual_seed(2)
    q, kr, vr, kt, vt = [torch.randn((1, n, h, 128), generator=g).bfloat16().cuda()
                         for n, h in ((1, 28), (3136, 4), (3136, 4), (97, 4), (97, 4))]
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


def test_captured_no_alloc_call_beside_its_contexts_other_calls():
    """A replayed allocation-free call on one stream, split attention and retrieval of the same context on another:
    they have no counters and no scratch in common."""
    g = torch.Generator().manual_seed(5)
    q, kr, vr, kt, vt = [torch.randn((1, n, h, 128), generator=g).bfloat16().to(DEV)
                         for n, h in ((1, 28), (12544, 4), (12544, 4), (97, 4), (97, 4))]
    qq, qk, qv = [torch.randn((1, 32, h, 128), generator=g).bfloat16().to(DEV) for h in (28, 4, 4)]
    table = torch.randn((200, 512), generator=g).to(DEV)
    r = Rekv(28, 4, 128, 196)
    want = r.decode_attention(q, kr, vr, kt, vt, 97)
    want_qa, want_idx = r.qa_attention(qq, kr, vr, qk, qv), r.retrieve_topk(table, 200, qq, 16)[0]
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
        got = [(r.qa_attention(qq, kr, vr, qk, qv), r.retrieve_topk(table, 200, qq, 16)[0]) for _ in range(10)]
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert all(torch.equal(a, want_qa) and torch.equal(i, want_idx) for a, i in got)


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
