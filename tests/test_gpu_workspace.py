"""Backwards and decodes in the least workspace a call takes (gist-phase segments of 16 query chunks, slices of 256 keys): the
results of the full-size workspace up to the grouping of fp32 sums, and nothing written behind the buffer."""
import pytest
import torch

import paper_2509_15763_amd as u
from paper_2509_15763_amd import synth
from test_gpu_decode_slices import _exact
from test_workspace import _decode_least_by_rule, _least_by_rule

pytestmark = pytest.mark.gpu


def _least(B, Hq, Hkv, L, D, r, W, S, mode):
    """Bytes for segments of 16 chunks, from a plan of shorter ones: a longer segment has the slots of its last part."""
    bp = u.unigist_bwd_plan_build(B, Hq, Hkv, L, D, r, W, S, mode)
    f = max(1, 16 // bp["seg_chunks"])
    tiles = [b - a for a, b in zip(bp["slot0"], bp["slot0"][1:])]
    merged = sum(tiles[min(len(tiles), i + f) - 1] for i in range(0, len(tiles), f))
    slots = bp["slot0"][-1]
    assert merged < slots, "a shape whose plan has nothing to give back"
    return bp["workspace_bytes"] - bp["partial_bytes"] // slots * (slots - merged)


def _guarded(n):
    buf = torch.full((n + 4096,), 255, dtype=torch.uint8, device="cuda")
    return buf[:n], buf[n:]


def _close(got, want):
    # fp32 sums of at most 32 partials in another grouping (2^-24 each) can move a bf16 result by 2^-8 in a share
    # 32 * 2^-24 / 2^-9 = 2^-10 of the elements: 2^-8 / sqrt(2^10) = 1.2e-4
    for a, b in zip(got, want):
        assert (a.float() - b.float()).norm() <= 3e-4 * b.float().norm()


@pytest.mark.parametrize("B,Hq,Hkv,L,D,r,W,S,mode", [
    (2, 32, 8, 2047, 128, 4, 128, 0, 0), (1, 4, 1, 4096, 128, 2, 64, 0, 0), (1, 8, 8, 3900, 64, 4, 333, 70, 0),
    (1, 8, 2, 3001, 96, 3, 20, 5, 1)])
def test_dense(B, Hq, Hkv, L, D, r, W, S, mode):
    q, k, v, do = (t.cuda() for t in synth.attn_inputs(B, Hq, Hkv, L, D, seed=L))
    kw = dict(sinks=S, window_mode=mode)
    out, lse = u.attn_fwd(q, k, v, r, W, **kw)
    want = u.attn_bwd(q, k, v, out, lse, do, r, W, **kw)
    ws, behind = _guarded(_least(B, Hq, Hkv, L, D, r, W, S, mode))
    _close(u.attn_bwd(q, k, v, out, lse, do, r, W, workspace=ws, **kw), want)
    ws.fill_(255)
    stages = tuple(torch.full_like(t, float("nan")) for t in (q, k, v))
    for stage in (1, 2, 4, 8, 16):
        u.attn_bwd(q, k, v, out, lse, do, r, W, workspace=ws, stages=stage, grads=stages, **kw)
    _close(stages, want)
    ws.fill_(255)
    t4 = lambda t: t.transpose(1, 2).contiguous().transpose(1, 2)
    _close(u.attn_bwd(t4(q), k, v, t4(out), lse, t4(do), r, W, workspace=ws, **kw), want)
    assert bool((behind == 255).all())


@pytest.mark.parametrize("docs", [[2047], [1500, 300] + [1111] * 6])  # four slices of the longest; the pack's own need
def test_pack(docs):
    Hq, Hkv, D, r, W = 8, 2, 128, 4, 128
    T, cu = sum(docs), [sum(docs[:i]) for i in range(len(docs) + 1)]
    q, k, v, do = (t[0].cuda() for t in synth.attn_inputs(1, Hq, Hkv, T, D, seed=T))
    out, lse = u.attn_fwd_varlen(q, k, v, r, W, cu)
    want = u.attn_bwd_varlen(q, k, v, out, lse, do, r, W, cu)
    pack, alone = (_least_by_rule(1, Hq, Hkv, d, D, r, W) for d in (docs, [max(docs)]))
    assert max(pack, 4 * alone) < u.unigist_attn_bwd_varlen_workspace(Hq, Hkv, T, D, r, W, cu, u.UNIGIST_BF16)
    ws, behind = _guarded(max(pack, 4 * alone))
    _close(u.attn_bwd_varlen(q, k, v, out, lse, do, r, W, cu, workspace=ws), want)
    assert bool((behind == 255).all())
    u.unigist_debug_force_plain_alu(1)  # the plain-ALU kernels work in the same buffer, a slice per stream
    try:
        plain = u.attn_bwd_varlen(q, k, v, out, lse, do, r, W, cu, workspace=ws)
        torch.cuda.synchronize()
    finally:
        u.unigist_debug_force_plain_alu(0)
    for a, b in zip(plain, want):
        assert (a.float() - b.float()).norm() <= 1e-2 * b.float().norm()  # two bf16 implementations
    assert bool((behind == 255).all())


@pytest.mark.parametrize("B,Hq,Hkv,Lk,D", [(8, 32, 8, 200, 128), (1, 8, 1, 1500, 64), (1, 34, 2, 500, 96)])
def test_decode(B, Hq, Hkv, Lk, D):
    gen = torch.Generator().manual_seed(Lk)
    q = torch.randn(B, Hq, D, generator=gen).bfloat16()
    k, v = (torch.randn(B, Hkv, Lk, D, generator=gen).bfloat16() for _ in range(2))
    n = [max(1, Lk - 60 * b) for b in range(B)]
    sl = torch.tensor(n, dtype=torch.int32).cuda()
    least = _decode_least_by_rule(B, Hq, Hkv, Lk, D, Hq // Hkv <= 15)
    assert least < u.unigist_decode_workspace(B, Hq, Hkv, Lk, D, u.UNIGIST_BF16)
    ws, behind = _guarded(least)
    o, l = _exact(q, k, v, n)
    # bf16 P and result: 2^-9 each on values of size at most max |v| <= 5, against float64
    out, lse = u.decode(q.cuda(), k.cuda(), v.cuda(), sl, workspace=ws)
    assert (out.cpu().double() - o).abs().max() <= 2e-2 and (lse.cpu().double() - l).abs().max() <= 1e-4
    ws.fill_(255)
    one = torch.ones(Hkv).cuda()
    k8, v8 = (u.quantize_e4m3(t.cuda(), one) for t in (k, v))
    wide = lambda c: c.cpu().view(torch.float8_e4m3fn).float()
    out, lse = u.decode_e4m3(q.cuda(), k8, v8, one, one, sl, workspace=ws)
    o, l = _exact(q, wide(k8), wide(v8), n)
    assert (out.cpu().double() - o).abs().max() <= 2e-2 and (lse.cpu().double() - l).abs().max() <= 1e-4
    assert bool((behind == 255).all())
