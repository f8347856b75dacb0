"""Retrieval at the edges of its kernels: tables around the one-pass rank's and the group-maximum selection's
limits, with equal scores; questions whose token rows and head groups do not fill the pooling kernel's
slots; the two scoring kernels on either side of their dispatch."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def reference(table, q, hkv):
    """Cosine of every frame vector with the mean query vector, in float64."""
    nt, hq, d = q.shape[-3:]
    m = q.reshape(nt, hkv, hq // hkv, d).mean(axis=(0, 2)).reshape(-1)
    return table @ m / (np.linalg.norm(table, axis=1) * np.linalg.norm(m))


def best(scores, k):
    """The k best by (score descending, frame ascending), in frame order."""
    return sorted(sorted(range(len(scores)), key=lambda f: (-scores[f], f))[:k])


@pytest.mark.parametrize("n_frames", [2, 63, 64, 65, 192, 255, 256, 257, 300, 4096, 4097])
@pytest.mark.parametrize("distinct", [1000000, 9])        # 9: nearly all scores are equal to others
def test_selection_on_its_own_scores(n_frames, distinct):
    from paper_2503_00540_amd.rekv import Rekv
    print(n_frames, distinct, flush=True)
    g = torch.Generator().manual_seed(n_frames)
    table = torch.randn((min(n_frames, distinct), 64), generator=g)
    table = table[torch.randint(0, table.shape[0], (n_frames,), generator=g)].contiguous().cuda()
    q = torch.randn((3, 5, 4, 64), generator=g).bfloat16().cuda()
    r = Rekv(4, 1, 64, 16, "bf16")
    for k in sorted({1, min(7, n_frames - 1), min(63, n_frames - 1), min(64, n_frames - 1), n_frames - 1, n_frames, n_frames + 3}):
        if k > 4096:
            continue
        # up to 256 frames: one launch for the first, a selection kernel of its own for the second
        for idx, n_sel, scores in (r.retrieve_topk(table, n_frames, q, k, want_scores=True),
                                   r.retrieve_external(table, q.float().mean(dim=(1, 2)), k, want_scores=True)):
            for i in range(3):
                n = min(k, n_frames)
                assert n_sel[i].item() == n
                assert idx[i].tolist() == best(scores[i].tolist(), n) + [-1] * (k - n)


@pytest.mark.parametrize("hq,hkv,d,dtype", [(14, 2, 64, "bf16"), (7, 1, 128, "bf16"), (3, 3, 36, "f32"), (71, 1, 4, "f32"), (8, 1, 256, "f32")])
@pytest.mark.parametrize("nt", [1, 9, 64, 147])
def test_pooling_and_scores(hq, hkv, d, dtype, nt):
    """fp32 sums of up to nt * G terms, dot products of hkv * d: 1e-5 covers a few dozen roundings of 6e-8."""
    from paper_2503_00540_amd.rekv import Rekv
    print(hq, hkv, d, dtype, nt, flush=True)
    g = torch.Generator().manual_seed(nt)
    table = torch.randn((37, hkv * d), generator=g)
    q = (torch.randn((2, nt, hq, d), generator=g) + 0.5).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    r = Rekv(hq, hkv, d, 16, dtype)
    _, _, scores = r.retrieve_topk(table.cuda(), 37, q.cuda(), 4, want_scores=True)
    for i in range(2):
        ref = reference(table.double().numpy(), q[i].double().numpy(), hkv)
        assert np.abs(scores[i].cpu().numpy() - ref).max() < 1e-5


@pytest.mark.parametrize("dim", [128, 132, 512, 1024, 1152])
@pytest.mark.parametrize("n_questions,n_frames", [(3, 33), (4, 33), (33, 65), (40, 3400)])   # the last above the line from 128 on
def test_external_scores_either_kernel(dim, n_questions, n_frames):
    from paper_2503_00540_amd.rekv import Rekv
    print(dim, n_questions, n_frames, flush=True)
    g = torch.Generator().manual_seed(dim)
    table, q = torch.randn((n_frames, dim), generator=g), torch.randn((n_questions, dim), generator=g)
    _, _, scores = Rekv(4, 1, 64, 16, "bf16").retrieve_external(table.cuda(), q.cuda(), 5, want_scores=True)
    t, m = table.double().numpy(), q.double().numpy()
    ref = m @ t.T / (np.linalg.norm(m, axis=1)[:, None] * np.linalg.norm(t, axis=1)[None])
    assert np.abs(scores.cpu().numpy() - ref).max() < 1e-5


@pytest.mark.parametrize("n_frames,b", [(1, 8), (7, 8), (8, 8), (9, 8), (41, 5), (12, 1)])
def test_short_last_block(n_frames, b):
    from paper_2503_00540_amd.rekv import Rekv
    table = torch.randn((n_frames, 128), generator=torch.Generator().manual_seed(b))
    got = Rekv(4, 2, 64, 16, "bf16").block_keys(table.cuda(), n_frames, b).cpu().double()
    ref = torch.stack([x.mean(dim=0) for x in table.double().split(b)])
    assert (got - ref).abs().max() < 1e-6


def test_short_retrieval_between_split_attention():
    """Both take their arrival counters from the same words, which every launch leaves at zero."""
    from paper_2503_00540_amd.rekv import Rekv
    from test_attention_plan import plan
    chosen = plan(28, 4, 128, 9, 40 * 49, 9, 2)
    assert chosen[0] == 1 and chosen[1] > 1
    g = torch.Generator().manual_seed(3)
    r = Rekv(28, 4, 128, 49, "bf16")
    table = torch.randn((200, 512), generator=g).cuda()
    q = torch.randn((2, 9, 28, 128), generator=g).bfloat16().cuda()
    kv = [torch.randn((2, n, 4, 128), generator=g).bfloat16().cuda() for n in (40 * 49, 40 * 49, 9, 9)]
    first = None
    for _ in range(4):
        got = [*r.retrieve_topk(table, 200, q, 11, want_scores=True), r.qa_attention(q, *kv)]
        torch.cuda.synchronize()
        first = first or [x.clone() for x in got]
        assert all(torch.equal(a, b) for a, b in zip(got, first))


def test_retrieval_captured_after_attention_needs_no_allocation():
    """The context's attention workspace serves a retrieval that is captured before it ever ran."""
    from paper_2503_00540_amd.rekv import Rekv
    g = torch.Generator().manual_seed(4)
    r = Rekv(28, 4, 128, 49, "bf16")
    table = torch.randn((700, 512), generator=g).cuda()
    q = torch.randn((2, 9, 28, 128), generator=g).bfloat16().cuda()
    kv = [torch.randn((2, n, 4, 128), generator=g).bfloat16().cuda() for n in (40 * 49, 40 * 49, 9, 9)]
    want = Rekv(28, 4, 128, 49, "bf16").retrieve_topk(table, 700, q, 11)
    r.qa_attention(q, *kv)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        got = r.retrieve_topk(table, 700, q, 11)
    torch.cuda.synchronize()
    for _ in range(3):
        got[0].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        r.qa_attention(q, *kv)
        torch.cuda.synchronize()
