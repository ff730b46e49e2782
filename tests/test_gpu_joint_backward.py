"""A short backward runs its gist phase, window phase and dQ as one launch and writes the gist rows of dK and dV in the
reduction behind it; run stage by stage it launches them one after the other.  Both against each other (and the joint one
against the oracle where it is small): padded head dimensions, sinks, unit windows, launches without a gist phase, gist
tiles that end inside the sequence.  On both sides of the rule that chooses, and with sinks and unit windows near it, one kv
head against float64: beyond the rule whole and staged backwards launch the same kernels."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_15763_amd as u
from paper_2509_15763_amd import synth
from _parity import TOL_GRAD_BF16, oracle_fwd_bwd, rel_l2, to_np

pytestmark = pytest.mark.gpu

#  B, Hq, Hkv, L, D, r, W, sinks, mode
SHAPES = [
    (1, 2, 1, 1, 64, 4, 8, 0, 0),           # one row
    (1, 4, 2, 300, 64, 4, 512, 0, 0),       # everything inside the window: no gist phase
    (2, 4, 1, 777, 128, 4, 64, 0, 0),
    (1, 7, 1, 1283, 96, 2, 33, 5, 0),       # padded columns, sinks, a group of seven
    (1, 4, 4, 1000, 48, 3, 100, 0, 0),
    (1, 8, 2, 1500, 128, 4, 20, 64, 1),     # window in units
    (2, 4, 2, 901, 64, 1, 16, 3, 1),
    (1, 1, 1, 1024, 64, 4, 128, 0, 0),
    (3, 16, 16, 3001, 64, 2, 70, 0, 0),     # segments of 32 chunks where separate launches take 16
    (1, 8, 8, 4100, 128, 4, 500, 3, 0),     # 16 and 4
]
LINE = [(1, 32, 8, 20480, 128, 16, 100, 0, 0), (1, 32, 8, 20481, 128, 16, 100, 0, 0),   # 5120 workgroups of dQ, the line with groups, and more
        (4, 32, 8, 6144, 64, 16, 64, 4, 0), (4, 32, 8, 6145, 64, 16, 64, 4, 0)]  # 6144, the line at D = 64, and more
LARGE = [(1, 32, 8, 12288, 128, 8, 256, 0, 0), (1, 32, 8, 12289, 128, 8, 256, 0, 0),  # 3072 workgroups of dQ, and more
         (1, 16, 16, 18432, 64, 16, 200, 0, 0), (1, 16, 16, 18561, 64, 16, 200, 0, 0)]  # 2304, 2336: D = 64, joint


@pytest.mark.parametrize("B,Hq,Hkv,L,D,r,W,S,mode", SHAPES + LARGE + LINE)
@pytest.mark.parametrize("strided", [False, True])
def test_whole_against_stages(B, Hq, Hkv, L, D, r, W, S, mode, strided):
    q, k, v, do = synth.attn_inputs(B, Hq, Hkv, L, D, seed=L)
    qd, kd, vd, dod = (t.cuda() for t in (q, k, v, do))
    kw = dict(sinks=S, window_mode=mode)
    out, lse = u.attn_fwd(qd, kd, vd, r, W, **kw)
    ws = torch.full((u.unigist_attn_bwd_workspace_ex(B, Hq, Hkv, L, D, r, W, S, mode, u.UNIGIST_BF16),), 255,
                    device="cuda", dtype=torch.uint8)  # NaNs: whatever is read must have been written
    want = tuple(torch.full_like(t, float("nan")) for t in (qd, kd, vd))
    for stage in (1, 2, 4, 8, 16):
        u.attn_bwd(qd, kd, vd, out, lse, dod, r, W, workspace=ws, stages=stage, grads=want, **kw)
    ws.fill_(255)
    if strided:
        t4 = lambda t: t.transpose(1, 2).contiguous().transpose(1, 2)
        got = u.attn_bwd(t4(qd), kd, vd, t4(out), lse, t4(dod), r, W, workspace=ws, **kw)
    else:
        got = tuple(torch.full_like(t, float("nan")) for t in (qd, kd, vd))
        u.attn_bwd(qd, kd, vd, out, lse, dod, r, W, workspace=ws, grads=got, **kw)
    assert torch.equal(got[0], want[0])
    # the same sums; one rounding of 2^-24 more where a gist row is put together can move a bf16 result by 2^-8 in one
    # of about 2^14 elements: 2^-8 / sqrt(2^14) = 3e-5
    for a, b in zip(got[1:], want[1:]):
        assert (a.float() - b.float()).norm() <= 3e-4 * b.float().norm() + 1e-6
    if L <= 1600 and L > 4:
        o, l, *grads = oracle_fwd_bwd(q, k, v, do, r, W, sinks=S, units=mode == 1)
        for a, b in zip(got, grads):
            assert rel_l2(to_np(a), b) <= TOL_GRAD_BF16


@pytest.mark.parametrize("strided", [False, True])
@pytest.mark.parametrize("onto", ["q", "dout", "out"])
@pytest.mark.parametrize("B,Hq,Hkv,L,D,r,W", [(2, 32, 8, 2047, 128, 4, 128), (1, 7, 1, 1283, 64, 2, 33),
                                              (13, 32, 8, 1601, 128, 8, 100)])  # 5304 workgroups of dQ: beyond the joint line
def test_dq_in_place_of_its_inputs(B, Hq, Hkv, L, D, r, W, onto, strided):
    # every row of q and dout is read by the two dK/dV phases as well, so dq has to be written behind them
    lay = (lambda t: t.transpose(1, 2).contiguous().transpose(1, 2)) if strided else (lambda t: t.contiguous())
    q, k, v, do = (t.cuda() for t in synth.attn_inputs(B, Hq, Hkv, L, D, seed=L))
    q, do = lay(q), lay(do)
    out, lse = u.attn_fwd(q, k, v, r, W)
    want = u.attn_bwd(q, k, v, out, lse, do, r, W)
    ws = torch.empty(u.unigist_attn_bwd_workspace(B, Hq, Hkv, L, D, r, W, u.UNIGIST_BF16), device="cuda", dtype=torch.uint8)
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    dq = {"q": q, "dout": do, "out": out}[onto]
    st = q.stride() if strided else (Hq * L * D, L * D, D)
    assert u.unigist_attn_bwd_strided(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), lse.data_ptr(), do.data_ptr(),
                                      dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), B, Hq, Hkv, L, D, r, W, 0, 0, *st[:3],
                                      u.UNIGIST_BF16, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(dq, want[0])
    # the same sums, put together in separate launches (as in test_whole_against_stages)
    for a, b in zip((dk, dv), want[1:]):
        assert (a.float() - b.float()).norm() <= 3e-4 * b.float().norm()


@pytest.mark.parametrize("onto", [None, "q", "dout", "out"])
def test_packed_dq_in_place_of_its_inputs(onto):
    # without overlap dQ runs first and computes delta itself; with it the delta pass runs first and dQ last
    Hq, Hkv, D, r, W, cu = 8, 2, 96, 4, 77, [0, 700, 701, 1500, 2111]
    q, k, v, do = (t[0].cuda() for t in synth.attn_inputs(1, Hq, Hkv, cu[-1], D, seed=3))
    out, lse = u.attn_fwd_varlen(q, k, v, r, W, cu)
    parts = []
    for a, b in zip(cu, cu[1:]):
        one = [t[None, :, a:b].contiguous() for t in (q, k, v, out, lse, do)]
        parts.append(u.attn_bwd(*one, r, W))
    want = [torch.cat(t, 2)[0] for t in zip(*parts)]
    ws = torch.empty(u.unigist_attn_bwd_varlen_workspace(Hq, Hkv, cu[-1], D, r, W, cu, u.UNIGIST_BF16), device="cuda", dtype=torch.uint8)
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    dq = {"q": q, "dout": do, "out": out}.get(onto, torch.empty_like(q))
    assert u.unigist_attn_bwd_varlen(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), lse.data_ptr(), do.data_ptr(),
                                     dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), Hq, Hkv, cu[-1], D, r, W, cu, u.UNIGIST_BF16,
                                     ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(dq, want[0])
    for a, b in zip((dk, dv), want[1:]):  # the same sums, grouped by the segments of the pack (as in test_whole_against_stages)
        assert (a.float() - b.float()).norm() <= 3e-4 * b.float().norm()


def _exact_group(q, k, v, do, r, W, S, mode):
    """Gradients of one kv head and its query heads (q, do [G, L, D], k, v [L, D] on the GPU) in float64, over row blocks."""
    G, L, D = q.shape
    q, k, v, do = (t.double() for t in (q, k, v, do))
    dq, dk, dv = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for i0 in range(0, L, 512):
        i1 = min(L, i0 + 512)
        seen = torch.from_numpy(oracle.mask_rows(np.arange(i0, i1), L, r, W, sinks=S, units=mode == 1)[:, :i1]).cuda()
        for g in range(G):
            p = ((q[g, i0:i1] @ k[:i1].T) / D ** 0.5).masked_fill_(~seen, float("-inf")).softmax(1)
            d = do[g, i0:i1]
            ds = p * (d @ v[:i1].T - (d * (p @ v[:i1])).sum(1, keepdim=True)) / D ** 0.5
            dv[:i1] += p.T @ d
            dq[g, i0:i1] = ds @ k[:i1]
            dk[:i1] += ds.T @ q[g, i0:i1]
    return dq, dk, dv


@pytest.mark.parametrize("B,Hq,Hkv,L,D,r,W,S,mode", [
    (1, 32, 8, 12288, 128, 8, 256, 0, 0), (1, 32, 8, 12289, 128, 8, 256, 0, 0),   # 3072 workgroups of dQ
    (1, 32, 8, 18432, 64, 16, 200, 0, 0), (1, 32, 8, 18433, 64, 16, 200, 0, 0),   # 4608
    (1, 32, 8, 12288, 128, 4, 30, 100, 1),                                        # sinks, window in units
    (2, 28, 4, 6000, 96, 4, 300, 70, 0),
    (1, 32, 8, 20480, 128, 8, 256, 0, 0), (1, 32, 8, 20481, 128, 8, 256, 0, 0),   # 5120: the line with groups of heads
    (4, 32, 8, 6144, 64, 16, 200, 0, 0), (4, 32, 8, 6145, 64, 16, 200, 0, 0),     # 6144: at D = 64
    (1, 32, 32, 12288, 128, 8, 256, 0, 0), (1, 32, 32, 12289, 128, 8, 256, 0, 0),  # 3072: the line without groups
    (1, 32, 32, 18432, 64, 16, 200, 0, 0), (1, 32, 32, 18433, 64, 16, 200, 0, 0),  # 4608: at D = 64
])
def test_both_sides_of_the_line_against_float64(B, Hq, Hkv, L, D, r, W, S, mode):
    q, k, v, do = (t.cuda() for t in synth.attn_inputs(B, Hq, Hkv, L, D, seed=L))
    kw = dict(sinks=S, window_mode=mode)
    out, lse = u.attn_fwd(q, k, v, r, W, **kw)
    dq, dk, dv = u.attn_bwd(q, k, v, out, lse, do, r, W, **kw)
    b, h, G = B - 1, Hkv - 2, Hq // Hkv
    heads = slice(h * G, (h + 1) * G)
    want = _exact_group(q[b, heads], k[b, h], v[b, h], do[b, heads], r, W, S, mode)
    got = dq[b, heads], dk[b, h][None], dv[b, h][None]
    for a, e in zip(got, (want[0], want[1][None], want[2][None])):
        for i0 in range(0, L, 128):  # tile by tile: a lost or doubled tile does not drown in the others
            x, y = a[:, i0:i0 + 128].double(), e[:, i0:i0 + 128]
            assert (x - y).norm() <= TOL_GRAD_BF16 * y.norm(), i0
    # a gist's column collects every segment's partial sums: the first ones on their own
    for c in range(min(64, (L - S) // (r + 1))):
        j = S + c * (r + 1) + r
        for a, e in ((dk, want[1]), (dv, want[2])):
            assert (a[b, h, j].double() - e[j]).norm() <= TOL_GRAD_BF16 * e[j].norm(), j
