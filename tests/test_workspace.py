"""The least workspace a backward takes: the one for gist-phase segments of 16 query chunks (32 in launches of many rounds),
which grows with the sequence up to that line, whatever shorter segments the plan of a large enough workspace has.  Probed through the
entry points with pointers that are never dereferenced: a call with too small a workspace is refused before anything is
launched, any other ends at the launch where there is no GPU."""
import pytest
import torch

import paper_2509_15763_amd as u

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="an accepted call would launch")
FAKE = 0x1000
EINVAL = 1


def _a(x):
    return (x + 255) & ~255


def _least_accepted(call, at_most):
    """Smallest workspace that `call` does not refuse."""
    lo, hi = 0, at_most
    while lo < hi:
        mid = (lo + hi) // 2
        lo, hi = (mid + 1, hi) if call(mid) == EINVAL else (lo, mid)
    return lo


def _sums(L, r, W, segc):
    """(slots, reduced tiles, chunk steps) per kv head for segments of segc chunks: a chunk c of 64 rows sees the gists left
    of its window's 128-key tile from afar, a segment has a slot for each 128 gists its last chunk sees."""
    NC = -(-L // 64)
    tiles = [-(-(max(0, 64 * c - min(W, L) + 1) // 128 * 128 // (r + 1)) // 128) for c in range(NC)]
    while -(-NC // segc) > 32:
        segc *= 2
    return sum(tiles[min(NC, s + segc) - 1] for s in range(0, NC, segc)), tiles[-1], sum(tiles)


def _least_by_rule(B, Hq, Hkv, docs, D, r, W):
    steps = sum(_sums(L, r, W, 16)[2] for L in docs) * B * Hkv
    segc = 32 if steps >= 512 * 32 * 5 else 16
    block = 2 * (64 if D <= 64 else 128) * 128 * 4
    part = sum(_sums(L, r, W, segc)[0] for L in docs) * B * Hkv * block
    comp = sum(_sums(L, r, W, segc)[1] for L in docs) * B * Hkv * block
    return 2 * _a(B * Hq * sum(docs) * 4) + part + comp


@pytest.mark.parametrize("B,Hq,Hkv,D,r,W", [(1, 32, 8, 128, 4, 512), (2, 32, 8, 128, 4, 128), (1, 8, 1, 64, 2, 64), (1, 28, 4, 96, 8, 900)])
def test_backward_takes_what_segments_of_16_need(B, Hq, Hkv, D, r, W):
    last = 0
    for L in list(range(1, 12000, 331)) + [2047, 3520, 3521, 4864, 4865, 8192, 8193, 32768, 70000]:
        shape = (B, Hq, Hkv, L, D, r, W, u.UNIGIST_BF16)
        query = u.unigist_attn_bwd_workspace(*shape)
        got = _least_accepted(lambda n: u.unigist_attn_bwd(*([FAKE] * 9), *shape, FAKE, n), query)
        assert got == _least_by_rule(B, Hq, Hkv, [L], D, r, W) <= query, L
        sd = (L * Hq * D, D, Hq * D)
        strided = lambda n: u.unigist_attn_bwd_strided(*([FAKE] * 9), B, Hq, Hkv, L, D, r, W, 0, 0, *sd, u.UNIGIST_BF16, FAKE, n)
        assert strided(got) != EINVAL and strided(got - 1) == EINVAL


@pytest.mark.parametrize("sinks,mode", [(0, 0), (70, 0), (5, 1)])
def test_a_buffer_for_the_longest_sequence_serves_the_shorter_ones(sinks, mode):
    W = 512 if mode == 0 else 100
    lengths = [100, 1024, 2047, 3000, 3520, 3521, 4000, 4864, 4865, 6000, 8192, 8193, 12000, 40000]
    for a, longer in enumerate(lengths):
        n = u.unigist_attn_bwd_workspace_ex(1, 32, 8, longer, 128, 4, W, sinks, mode, u.UNIGIST_BF16)
        for L in lengths[:a + 1]:
            assert u.unigist_attn_bwd_ex(*([FAKE] * 9), 1, 32, 8, L, 128, 4, W, sinks, mode, u.UNIGIST_BF16, FAKE, n, 31) != EINVAL


@pytest.mark.parametrize("docs", [[2047], [300, 4096, 1, 5000], [3520] * 3, [8193, 100], [1024] * 70, [32768]])
def test_packs(docs):
    Hq, Hkv, D, r, W = 32, 8, 128, 4, 512
    cu = [sum(docs[:i]) for i in range(len(docs) + 1)]
    query = u.unigist_attn_bwd_varlen_workspace(Hq, Hkv, cu[-1], D, r, W, cu, u.UNIGIST_BF16)
    call = lambda n: u.unigist_attn_bwd_varlen(*([FAKE] * 9), Hq, Hkv, cu[-1], D, r, W, cu, u.UNIGIST_BF16, FAKE, n)
    got = _least_accepted(call, query)
    # the pack's own need, or four slices for its longest document taken alone
    alone = max(_least_by_rule(1, Hq, Hkv, [L], D, r, W) for L in docs)
    assert got == max(_a(_least_by_rule(1, Hq, Hkv, docs, D, r, W)), 4 * _a(alone)) <= query


def _decode_least_by_rule(B, Hq, Hkv, Lk, D, grouped):
    """Slices of at least 256 keys, in rounds of 256 workgroups."""
    units = B * (Hkv if grouped else Hq)
    target = 256 if units <= 64 else 512 if units <= 256 else 1024
    most = max(1, min(64, max(4, -(-target // units)), -(-Lk // 256)))
    cost = lambda n: -(-units * n // 256) * 256 / (units * n) * (1 + 0.01 * n) * (1.05 if units * n < target else 1.0)
    n = min(range(1, most + 1), key=cost)
    return _a(B * Hq * n * ((64 if D <= 64 else 128) + 2) * 4)


@pytest.mark.parametrize("Hq,Hkv,D", [(32, 8, 128), (8, 1, 64), (16, 16, 96), (34, 2, 128)])  # the last: the vector kernel
@pytest.mark.parametrize("Lk", [1, 129, 200, 500, 1500, 9001])
def test_decode_takes_what_slices_of_256_keys_need(Hq, Hkv, D, Lk):
    sizes = []
    for B in range(1, 40):
        query = u.unigist_decode_workspace(B, Hq, Hkv, Lk, D, u.UNIGIST_BF16)
        call = lambda n: u.unigist_decode(*([FAKE] * 4), None, B, Hq, Hkv, Lk, None, D, u.UNIGIST_BF16, FAKE, n)
        call8 = lambda n: u.unigist_decode_e4m3(*([FAKE] * 6), None, B, Hq, Hkv, Lk, None, D, FAKE, n)
        least = _decode_least_by_rule(B, Hq, Hkv, Lk, D, Hq // Hkv <= 15)
        assert _least_accepted(call, query) == least <= query
        assert call8(least) != EINVAL and call8(least - 1) == EINVAL
        sizes.append((query, least))
    if (Hq, Hkv, Lk) == (32, 8, 200):
        # one slice of 256 keys per sequence from 9 sequences on: a buffer for any of those batches serves 8
        assert all(sizes[7][1] <= q < sizes[7][0] for q, _ in sizes[8:12])


@pytest.mark.parametrize("Hq,Hkv,D", [(32, 8, 128), (120, 8, 128), (8, 1, 64), (16, 16, 96)])
def test_additional_slices_keep_within_the_built_in_array(Hq, Hkv, D):
    """Long slabs ask for more slices than the rule for shorter ones, up to the size of the built-in array where those fit it: what it
    serves does not depend on them, and an array and a workspace of the size asked for hold the same slices."""
    scratch = u.unigist_decode_noalloc_scratch_bytes()
    more = 0
    for B in (8, 12, 20, 24, 36, 40, 64, 65, 68, 100, 120, 128, 250, 500, 1000):
        base = lambda Lk: u.unigist_decode_workspace(B, Hq, Hkv, Lk, D, u.UNIGIST_BF16)
        for Lk in (8192, 12000, 17408, 40000):
            if base(8191) > scratch:  # the slices of a shorter slab, as many
                assert u.unigist_decode_noalloc(*([FAKE] * 4), None, B, Hq, Hkv, Lk, None, D, u.UNIGIST_BF16) == 4
            else:
                assert base(Lk) <= scratch
                assert u.unigist_decode_noalloc(*([FAKE] * 4), None, B, Hq, Hkv, Lk, None, D, u.UNIGIST_BF16) != 4
            assert base(Lk) >= base(8191)
            more += base(Lk) > base(8191)
    assert more


@pytest.mark.parametrize("B,Hq,Hkv,Lk,D,slices", [
    (64, 32, 8, 17408, 128, 4), (32, 32, 8, 17408, 128, 4), (16, 32, 8, 17408, 128, 4), (128, 32, 8, 17408, 128, 3),  # whole rounds; what the built-in array holds
    (64, 32, 8, 12000, 128, 6), (32, 32, 8, 16383, 128, 6), (32, 32, 8, 16384, 128, 4), (64, 16, 4, 16384, 64, 6), (64, 16, 4, 16383, 64, 2),
    (16, 32, 8, 12000, 128, 6), (48, 32, 8, 12000, 128, 6), (128, 32, 8, 12000, 128, 2), (192, 32, 8, 9000, 64, 2),   # six for two to four, two for one
    (100, 8, 1, 30000, 128, 5), (90, 32, 8, 10000, 128, 2), (125, 32, 8, 10000, 128, 2), (100, 8, 1, 12000, 128, 5),  # kept
    (21, 32, 8, 16383, 128, 6), (21, 32, 8, 16384, 128, 6),
    (8, 32, 8, 8192, 128, 8), (10, 32, 8, 9000, 128, 6), (13, 32, 8, 9000, 128, 4), (18, 32, 8, 9000, 128, 7), (12, 32, 8, 9000, 96, 8),
    (44, 32, 8, 9000, 128, 8), (60, 32, 8, 9000, 64, 4), (1000, 32, 8, 17408, 128, 2)])
def test_slices_of_long_slabs_fill_rounds_of_workgroups(B, Hq, Hkv, Lk, D, slices):
    assert u.unigist_decode_workspace(B, Hq, Hkv, Lk, D, u.UNIGIST_BF16) == _a(B * Hq * slices * ((64 if D <= 64 else 128) + 2) * 4)
