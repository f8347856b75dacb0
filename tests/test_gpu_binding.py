"""The native half of the binding against the Python methods: ordinary calls are taken and launch the same; every other
form ends as it does without it - served, or refused with the same error."""
import numpy as np
import pytest
import torch

from paper_2503_00540_amd import rekv
from paper_2503_00540_amd.rekv import Rekv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class PythonOnly:
    """In the place of the native half: leaves every call to the Python method."""
    def __getattr__(self, name):
        return lambda *a: None


class Counting:
    """Counts the calls that the native half takes."""
    def __init__(self, inner):
        self.inner, self.taken = inner, 0

    def __getattr__(self, name):
        def call(*a):
            r = getattr(self.inner, name)(*a)
            self.taken += r is not None
            return r
        return call


HQ, HKV, D, NF, F = 8, 2, 64, 6, 20


def setup():
    g = torch.Generator().manual_seed(3)
    mk = lambda *s, dt=torch.bfloat16: torch.randn(s, generator=g).to(dt).to(DEV)
    t = {"q": mk(2 * 7, HQ, D), "k": mk(F * NF, HKV, D), "v": mk(F * NF, HKV, D), "qq": mk(2, 5, HQ, D), "kq": mk(2, 9, HKV, D),
         "vq": mk(2, 9, HKV, D), "table": mk(F, HKV * D, dt=torch.float32), "emb": mk(F, 32, dt=torch.float32), "qe": mk(2, 32, dt=torch.float32),
         "idx": torch.tensor([[1, 4, 5], [0, 7, 19]], dtype=torch.int32, device=DEV), "n_sel": torch.tensor([3, 2], dtype=torch.int32, device=DEV)}
    t["kr"], t["vr"] = mk(2, 3 * NF, HKV, D), mk(2, 3 * NF, HKV, D)
    return t


def calls(t, r):
    """Ordinary calls of every method."""
    e = torch.empty_like
    i = t["idx"]
    return {
        "encode": lambda: r.encode_chunk(t["q"], t["k"], t["v"], 30, 7, 2, 25),
        "encode out": lambda: r.encode_chunk(t["q"], t["k"], t["v"], 30, 7, 2, 25, out=e(t["q"])),
        "frame_keys": lambda: r.frame_keys(t["k"], F),
        "frame_keys out": lambda: r.frame_keys(t["k"], 3, out=torch.zeros(5, HKV * D, device=DEV)),
        "retrieve": lambda: r.retrieve_topk(t["table"], F, t["qq"], 3, want_scores=True),
        "retrieve tables": lambda: r.retrieve_topk(torch.stack([t["table"], t["table"] * 2 + 1]), F, t["qq"], 4, frame_keys_stride=F * HKV * D)[:2],
        "external": lambda: r.retrieve_external(t["emb"], t["qe"], 4, tau=0.5, want_scores=True),
        "blocks": lambda: r.block_keys(t["table"], 19, 4),
        "blocks out": lambda: r.block_keys(t["table"], 19, 4, out=torch.zeros(6, HKV * D, device=DEV)),
        "expand": lambda: r.expand_blocks(i, 4, 19),
        "gather": lambda: r.gather_kv(t["k"], t["v"], i),
        "gather dst": lambda: r.gather_kv(t["k"], t["v"], i, n_src_frames=6, dst_k=e(t["kr"]), dst_v=e(t["vr"])),
        "layers": lambda: r.gather_kv_layers([t["k"], t["v"]], [t["v"], t["k"]], i.view(2, 1, 3)),
        "rope": lambda: r.gather_kv_rope(t["k"], t["v"], i, pos_offset=3, mode="static", src_rotated=True, layout="interleaved", base=500.0),
        "qa": lambda: r.qa_attention(t["qq"], t["kr"], t["vr"], t["kq"][:, :5].contiguous(), t["vq"][:, :5].contiguous(), n_sel=t["n_sel"]),
        "decode": lambda: r.decode_attention(t["qq"], t["kr"], t["vr"], t["kq"], t["vq"], 8, n_sel=t["n_sel"]),
        "decode no_alloc": lambda: r.decode_attention(t["qq"], t["kr"], t["vr"], t["kq"], t["vq"], 8, out=e(t["qq"]), no_alloc=True),
        "indexed": lambda: r.attention_indexed(t["qq"], t["k"], t["v"], i, 2, t["kq"], t["vq"], 9, n_sel=t["n_sel"]),
        "indexed rope": lambda: r.attention_indexed_rope(t["qq"], t["k"], t["v"], i, t["kq"], t["vq"], 9, n_src_frames=F, n_sel=t["n_sel"], k_pos=e(t["kr"])),
    }


def same(a, b):
    if isinstance(a, (tuple, list)):
        return type(a) is type(b) and len(a) == len(b) and all(same(x, y) for x, y in zip(a, b))
    if a is None or b is None:
        return a is b
    return a.dtype == b.dtype and a.shape == b.shape and a.device == b.device and torch.equal(a, b)


def outcome(call):
    try:
        return call()
    except Exception as e:
        return type(e).__name__, str(e)


def test_ordinary_calls_are_taken_and_launch_the_same():
    t, r = setup(), Rekv(HQ, HKV, D, NF)
    native = r._fast
    for name, call in calls(t, r).items():
        r._fast = Counting(native)
        got = call()
        assert r._fast.taken == 1, name
        r._fast = PythonOnly()
        want = call()
        if name == "frame_keys out":
            got, want = got[:3], want[:3]
        assert same(got, want), name
    r._fast = native


def test_given_outputs_are_returned():
    t, r = setup(), Rekv(HQ, HKV, D, NF)
    out, dk, dv = torch.empty_like(t["q"]), torch.empty_like(t["kr"]), torch.empty_like(t["vr"])
    assert r.encode_chunk(t["q"], t["k"], t["v"], 0, 7, 2, 25, out=out) is out
    got = r.gather_kv(t["k"], t["v"], t["idx"], dst_k=dk, dst_v=dv)
    assert got[0] is dk and got[1] is dv


def test_unusual_and_refused_calls_end_as_without_it():
    t, r = setup(), Rekv(HQ, HKV, D, NF)
    i = t["idx"]
    strided = torch.stack([i, i], dim=-1)[..., 0]
    forms = {
        "short cache": lambda: r.encode_chunk(t["q"], t["k"], t["v"], 1000, 7, 2, 25),
        "negative token": lambda: r.encode_chunk(t["q"], t["k"], t["v"], -1, 7, 2, 25),
        "huge token": lambda: r.encode_chunk(t["q"], t["k"], t["v"], 1 << 70, 7, 2, 25),
        "float size": lambda: r.encode_chunk(t["q"], t["k"], t["v"], 0, 7.0, 2, 25),
        "numpy size": lambda: r.encode_chunk(t["q"], t["k"], t["v"], 0, np.int64(7), 2, 25),
        "wrong dtype": lambda: r.encode_chunk(t["q"].float(), t["k"], t["v"], 0, 7, 2, 25),
        "host tensor": lambda: r.encode_chunk(t["q"].cpu(), t["k"], t["v"], 0, 7, 2, 25),
        "not contiguous": lambda: r.encode_chunk(t["q"].transpose(0, 1).contiguous().transpose(0, 1), t["k"], t["v"], 0, 7, 2, 25),
        "no tensor": lambda: r.encode_chunk(None, t["k"], t["v"], 0, 7, 2, 25),
        "misaligned": lambda: r.frame_keys(torch.zeros(NF * HKV * D + 1, dtype=torch.bfloat16, device=DEV)[1:].view(NF, HKV, D), 1),
        "no frames": lambda: r.frame_keys(t["k"], 0),
        "negative frames": lambda: r.frame_keys(t["k"], -1),
        "small table": lambda: r.frame_keys(t["k"], 3, out=torch.zeros(2, HKV * D, device=DEV)),
        "k = 0": lambda: r.retrieve_topk(t["table"], F, t["qq"], 0),
        "odd stride": lambda: r.retrieve_topk(t["table"], 4, t["qq"], 2, frame_keys_stride=515),
        "negative stride": lambda: r.retrieve_topk(t["table"], F, t["qq"], 3, frame_keys_stride=-4),
        "int tau": lambda: r.retrieve_external(t["emb"], t["qe"], 4, tau=2),
        "zero tau": lambda: r.retrieve_external(t["emb"], t["qe"], 4, tau=0.0),
        "b = 0": lambda: r.block_keys(t["table"], F, 0),
        "strided blocks": lambda: r.expand_blocks(strided, 4, 19),
        "strided idx": lambda: r.gather_kv(t["k"], t["v"], strided),
        "long idx": lambda: r.gather_kv(t["k"], t["v"], i.long()),
        "wrong dst": lambda: r.gather_kv(t["k"], t["v"], i, dst_k=torch.empty_like(t["k"])),
        "more frames than there are": lambda: r.gather_kv(t["k"], t["v"], i, n_src_frames=F + 1),
        "no frames in the arena": lambda: r.gather_kv(t["k"], t["v"], i, n_src_frames=0),
        "tuple of layers": lambda: r.gather_kv_layers((t["k"], t["v"]), (t["v"], t["k"]), i.view(2, 1, 3)),
        "no layers": lambda: r.gather_kv_layers([], [], i.view(2, 1, 3)[:0]),
        "too many layers": lambda: r.gather_kv_layers([t["k"]] * 65, [t["v"]] * 65, torch.zeros((65, 1, 1), dtype=torch.int32, device=DEV)),
        "unknown mode": lambda: r.gather_kv_rope(t["k"], t["v"], i, mode="other"),
        "int base": lambda: r.gather_kv_rope(t["k"], t["v"], i, base=10000),
        "int flag": lambda: r.gather_kv_rope(t["k"], t["v"], i, src_rotated=1),
        "nothing retrieved": lambda: r.qa_attention(t["qq"], t["kr"][:, :0], t["vr"][:, :0], t["kq"][:, :5].contiguous(), t["vq"][:, :5].contiguous()),
        "n_sel of another length": lambda: r.qa_attention(t["qq"], t["kr"], t["vr"], t["kq"][:, :5].contiguous(), t["vq"][:, :5].contiguous(), n_sel=t["n_sel"][:1]),
        "text shorter than the new tokens": lambda: r.decode_attention(t["qq"], t["kr"], t["vr"], t["kq"], t["vq"], 3),
        "text longer than its cache": lambda: r.decode_attention(t["qq"], t["kr"], t["vr"], t["kq"], t["vq"], 10),
        "int no_alloc": lambda: r.decode_attention(t["qq"], t["kr"], t["vr"], t["kq"], t["vq"], 8, no_alloc=1),
        "parameter": lambda: r.decode_attention(torch.nn.Parameter(t["qq"]).detach(), t["kr"], t["vr"], t["kq"], t["vq"], 8),
        "wrong out": lambda: r.attention_indexed(t["qq"], t["k"], t["v"], i, 2, t["kq"], t["vq"], 9, out=t["q"]),
        "wrong k_pos": lambda: r.attention_indexed_rope(t["qq"], t["k"], t["v"], i, t["kq"], t["vq"], 9, k_pos=t["k"]),
    }
    native = r._fast
    for name, call in forms.items():
        print(name, flush=True)
        r._fast = native
        got = outcome(call)
        r._fast = PythonOnly()
        want = outcome(call)
        assert (got == want) if isinstance(want[0], str) else same(got, want), (name, got, want)
    r._fast = native
    r.close()
    assert outcome(lambda: r.frame_keys(t["k"], 1))[0] == "RekvError"


def test_a_tensor_that_gives_no_address_is_refused():
    """Its address throws: the native half leaves the call, with the interpreter as it was, to the Python method."""
    t, r = setup(), Rekv(HQ, HKV, D, NF)
    want = r.frame_keys(t["k"], F)
    sealed = t["k"].clone()
    torch._C._set_throw_on_mutable_data_ptr(sealed)
    for call in (lambda: r.frame_keys(sealed, F), lambda: r.encode_chunk(t["q"], sealed, t["v"], 30, 7, 2, 25),
                 lambda: r.gather_kv(sealed, t["v"], t["idx"]), lambda: r.gather_kv_layers([t["k"], sealed], [t["v"], t["k"]], t["idx"].view(2, 1, 3))):
        with pytest.raises(RuntimeError):
            call()
    assert torch.equal(r.frame_keys(t["k"], F), want)


def test_calls_without_the_native_half_end_alike(monkeypatch):
    """Where _binding.so does not load, the Python methods serve every ordinary call."""
    t, r = setup(), Rekv(HQ, HKV, D, NF)
    want = {name: call() for name, call in calls(t, r).items()}
    monkeypatch.setattr(rekv, "_native", rekv._NoNative)
    plain = Rekv(HQ, HKV, D, NF)
    for name, call in calls(t, plain).items():
        got, ref = call(), want[name]
        if name == "frame_keys out":
            got, ref = got[:3], ref[:3]
        assert same(got, ref), name
