"""Shapes whose launches are too small to fill the chip: the backward's gist phase then runs in shorter segments
(2, 4 or 8 query chunks instead of 16 and more), up to the 32 segments a plan can carry."""
import pytest
import torch

import paper_2509_15763_amd as u
from paper_2509_15763_amd import synth
from _parity import check_kv_group

#  B, Hq, Hkv, L, r, W, segment length the plan takes
SHAPES = [
    (1, 1, 1, 1024, 4, 128, 2),     # one head
    (1, 4, 1, 4096, 2, 64, 2),      # 64 chunks in 32 segments of 2: as many as a plan carries
    (1, 4, 2, 4100, 2, 64, 4),      # ... and one chunk more: the length doubles
    (2, 8, 8, 3003, 4, 100, 4),     # ragged last chunk
    (2, 8, 8, 3900, 4, 333, 8),
    (1, 8, 8, 8191, 4, 1024, 8),
]


@pytest.mark.parametrize("B,Hq,Hkv,L,r,W,segc", SHAPES)
def test_segment_length_of_the_plan(B, Hq, Hkv, L, r, W, segc):
    bp = u.unigist_bwd_plan_build(B, Hq, Hkv, L, 128, r, W)
    assert bp["seg_chunks"] == segc and bp["n_segs"] == -(-bp["n_chunks"] // segc) <= 32
    assert bp["workspace_bytes"] == u.unigist_attn_bwd_workspace(B, Hq, Hkv, L, 128, r, W, u.UNIGIST_BF16)


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,L,r,W,segc", SHAPES[:5])
def test_gradients_against_the_oracle(B, Hq, Hkv, L, r, W, segc):
    q, k, v, do = synth.attn_inputs(B, Hq, Hkv, L, 128, seed=L)
    qd, kd, vd, dod = (t.cuda() for t in (q, k, v, do))
    out, lse = u.attn_fwd(qd, kd, vd, r, W)
    grads = u.attn_bwd(qd, kd, vd, out, lse, dod, r, W)
    res = tuple(t.cpu() for t in (out, lse) + grads)
    check_kv_group("small launch", q, k, v, do, res, B - 1, Hkv - 1, r, W)
