"""The plan of a bf16 attention launch (which kernel, how many splits of the key range), without a GPU: what the
chosen launch needs stays within what the kernel has, over the whole argument range."""
import ctypes
import math
import random

import pytest

from paper_2503_00540_amd import rekv


def plan(hq, hkv, d, len_q, len_a, len_b, items=1, encode=False, first=1 << 40, in_place=False):
    """(row waves per workgroup or 0 for the 128-row kernel, splits, row blocks, workspace bytes, reserved bytes)"""
    f = rekv.lib().rekv_internal_attention_plan
    f.restype = None
    f.argtypes = [ctypes.c_int32] * 4 + [ctypes.c_int64] + [ctypes.c_int32] * 5 + [ctypes.c_void_p]
    out = (ctypes.c_int64 * 5)()
    f(hq, hkv, d, int(encode), first, items, len_q, len_a, len_b, int(in_place), out)
    return tuple(out)


def key_groups(hq, hkv, d, len_q, len_a, len_b, items=1, encode=False, first=1 << 40, in_place=False):
    f = rekv.lib().rekv_internal_attention_key_groups
    f.restype = ctypes.c_int32
    f.argtypes = [ctypes.c_int32] * 4 + [ctypes.c_int64] + [ctypes.c_int32] * 5
    return f(hq, hkv, d, int(encode), first, items, len_q, len_a, len_b, int(in_place))


def last_arriver_lds(rows, d):
    """Bytes that the merge of a row block of so many rows lays over the tiles: of all thread groups but the first, the partial
    sums from the front, their maxima and sums behind the room that the most of those can take."""
    per = -(-(rows * d // 4) // 64) * 64
    groups = 512 // per if per * 2 <= 512 else 1
    assert (groups - 1) * per <= 512 - 64
    return (512 - 64) * 16 + (groups - 1) * per * 8 if groups > 1 else 0


def workspace_of_128_row_blocks(hq, hkv, d, len_q, len_a, len_b, items):
    """What a context holds after a call, whichever kernel takes it: the partial results of splitting 128-row workgroups
    over the keys (512 of them in all, each with at least 8 tiles of 32 keys, 2 where it has at most 32 rows)."""
    m_rows = len_q * (hq // hkv)
    row_blocks = -(-m_rows // 128)
    base = items * hkv * row_blocks
    tiles = -(-len_a // 32) + -(-len_b // 32)
    splits = max(1, min(512 // base, tiles // (2 if m_rows <= 32 else 8))) if base < 512 else 1
    return base * splits * 128 * (d + 2) * 4 if splits > 1 else 0


def shapes():
    # one KV head, few rows, long context: where the split count is largest
    for hq in (1, 2, 3, 8, 16):
        for len_q in (1, 2, 3, 31, 32, 33, 65):
            for len_a in range(800_000, 1_060_000, 9_973):
                for d in (64, 128):
                    yield hq, 1, d, len_q, len_a, len_q, 1, len_a % 2 == 0
    rng = random.Random(7)
    log_int = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    for _ in range(60_000):
        hkv, len_q, encode = rng.choice([1, 1, 2, 4, 8]), log_int(1, 4000), rng.random() < 0.5
        yield (hkv * rng.choice([1, 2, 3, 5, 7, 8, 16]), hkv, rng.choice([64, 128]), len_q, log_int(1, 1 << 22),
               len_q if encode else len_q + rng.choice([0, log_int(1, 4000)]), log_int(1, 600), encode)


def test_split_launches_fit_their_kernel():
    n_split = n_two = 0
    for hq, hkv, d, len_q, len_a, len_b, items, encode in shapes():
        wave, splits, row_blocks, ws, reserved = plan(hq, hkv, d, len_q, len_a, len_b, items, encode)
        where = (hq, hkv, d, len_q, len_a, len_b, items, encode)
        assert wave in (0, 1, 2) and splits >= 1, where
        assert ws <= 33 << 20, where                              # the allocation-free entry point's scratch
        assert reserved == workspace_of_128_row_blocks(hq, hkv, d, len_q, len_a, len_b, items), where
        assert ws <= reserved, where
        groups = key_groups(hq, hkv, d, len_q, len_a, len_b, items, encode)
        assert groups in (1, 2) and (groups == 1 or not wave), where
        if not wave:
            blocks = items * hkv * row_blocks
            assert row_blocks == -(-len_q * (hq // hkv) // 128), where
            assert ws == (blocks * splits * 128 * (d + 2) * 4 if splits > 1 else 0), where
            if groups == 2:                                       # arrival counters, one resident workgroup per CU
                n_two += 1
                assert blocks * splits <= 256 and len_q * (hq // hkv) > 32, where
            continue
        m_rows, t = len_q * (hq // hkv), 32 * wave
        assert row_blocks == -(-m_rows // t), where
        assert items * hkv * row_blocks * splits <= 512, where    # arrival counters, resident workgroups
        if splits == 1:
            assert ws == 0, where
            continue
        n_split += 1
        assert ws >= items * hkv * row_blocks * splits * t * (d + 2) * 4, where
        last = m_rows - (row_blocks - 1) * t
        assert max(last_arriver_lds(rows, d) for rows in {last, min(m_rows, t)}) <= 8 * 2 * 32 * d * 2, where
        assert splits * t <= (7296 if d == 64 else 15488), where      # the most that were ever measured
    assert n_split > 1000 and n_two > 1000


@pytest.mark.parametrize("hq,hkv,d,l_x,items", [(8, 2, 128, 66, 1), (28, 4, 128, 196, 1), (14, 2, 64, 144, 2), (16, 8, 64, 392, 1)])
@pytest.mark.parametrize("past", [0, 66, 1000])
def test_a_window_counts_as_far_as_the_stream_reaches(hq, hkv, d, l_x, items, past):
    """A window that is not full is split like one of the stream's length, not for tiles that do not exist."""
    reach = past + (items - 1) * l_x
    chosen = plan(hq, hkv, d, l_x, 15_000, l_x, items, True, past)
    assert chosen[0] > 0
    assert chosen[1] <= max(1, -(-(-(-reach // 32) + -(-l_x // 32)) // (8 // chosen[0])))
    assert chosen[:4] == plan(hq, hkv, d, l_x, 1 << 24, l_x, items, True, past)[:4]


@pytest.mark.parametrize("d,hq,hkv,len_q", [(64, 16, 8, 25), (128, 64, 8, 1), (64, 14, 2, 1)])
def test_beyond_the_last_level_cache_the_128_row_kernel(d, hq, hkv, len_q):
    for len_a in (4000, 8000, 20_000):
        items = -(-270_000_000 // (len_a * hkv * d * 4))
        assert plan(hq, hkv, d, len_q, len_a, len_q, items)[0] == 0


@pytest.mark.parametrize("hq,hkv,d,len_q,len_a,encode", [
    (16, 8, 64, 392, 60 * 196, True),        # 39 us with 128-row workgroups and K and V from HBM, 64 without
    (16, 8, 64, 392, 49 * 196, True),
])
def test_launches_that_splitting_the_keys_slows_down(hq, hkv, d, len_q, len_a, encode):
    assert plan(hq, hkv, d, len_q, len_a, len_q, 1, encode)[0] == 0


@pytest.mark.parametrize("hq,hkv,d,len_q,len_a,len_b,items,wave", [
    # head_dim 64, more users than half of the chip's places: an unsplit 128-row workgroup has rows for one wavefront of four
    (14, 2, 64, 1, 237, 275, 144, 1),        # us, replayed from a graph: 10.1 and 12.4 with 128-row workgroups
    (14, 2, 64, 1, 819, 75, 219, 1),         # 17.0 and 18.9
    (16, 8, 64, 1, 163, 122, 37, 1),         # 8.1 and 9.7
    (28, 4, 64, 1, 1512, 104, 104, 1),       # 30.0 and 32.7
    # a few hundred keys of one user: one launch
    (28, 4, 128, 1, 193, 70, 1, 1),          # 6.2 and 7.7
    (14, 2, 64, 4, 137, 224, 1, 1),          # 5.3 and 7.1
    # around a thousand keys, or many of many users: 128-row workgroups split over the keys and a merge
    (8, 4, 128, 1, 467, 35, 3, 0),           # 8.2 and 9.8 with the split-key kernel
    (64, 8, 128, 1, 1008, 13, 1, 0),         # 8.4 and 9.7
    (8, 2, 128, 1, 720, 30, 5, 0),
    (64, 8, 128, 1, 1152, 30, 1, 0),
    (32, 32, 64, 1, 4716, 28, 5, 0),         # 36 and 48
])
def test_few_rows_take_the_faster_kernel(hq, hkv, d, len_q, len_a, len_b, items, wave):
    assert plan(hq, hkv, d, len_q, len_a, len_b, items)[0] == wave


def test_frames_in_place_are_judged_like_gathered_ones():
    """With more than 32 rows, except beyond 268 MB of listed K and V at head_dim 64, where questions share what they list.  With
    fewer a call that splits 128-row workgroups in place does so gathered as well."""
    rng, beyond, few = random.Random(11), 0, 0
    log_int = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    for _ in range(60_000):
        hkv, d, len_q, items, frames = rng.choice([1, 2, 4, 8, 16]), rng.choice([64, 128]), log_int(1, 300), log_int(1, 300), log_int(1, 1024)
        hq, len_a, len_b = hkv * rng.choice([1, 2, 3, 7, 8]), frames * rng.choice([33, 144, 196, 256]), len_q + rng.choice([0, log_int(1, 300)])
        where = hq, hkv, d, len_q, len_a, len_b, items
        gathered, in_place = [plan(*where, in_place=x) for x in (False, True)]
        if len_q * (hq // hkv) <= 32:
            assert gathered == in_place or (gathered[0], in_place[0]) == (0, 1), where
            few += gathered != in_place
            continue
        large = d == 64 and items * (len_a + len_b) * hkv * d * 4 > 268_000_000
        assert gathered == in_place or large, where
        beyond += gathered != in_place
    assert beyond > 100 and few > 100


@pytest.mark.parametrize("hq,hkv,d,len_q,len_a,len_b,items", [
    (28, 4, 128, 1, 1683, 41, 2),            # us, replayed from a graph: 9.4 and 10.7 with 128-row workgroups
    (64, 8, 128, 1, 747, 21, 1),             # 9.1 and 9.9
    (14, 2, 64, 1, 6076, 35, 48),            # 24.0 and 27.3
    (28, 4, 128, 1, 2156, 23, 41),           # 32.0 and 35.7
])
def test_few_rows_in_place_take_the_faster_kernel(hq, hkv, d, len_q, len_a, len_b, items):
    assert plan(hq, hkv, d, len_q, len_a, len_b, items, in_place=True)[0] == 1
