"""The row-side kernels (forward, dQ, prefill) split a kv head's work into units of 32 rows of one query head, four
to a workgroup: group sizes that divide four, that are divided by it and that do neither, with row counts around the
edges of a unit, so that workgroups span row blocks and the last one has waves without a unit."""
import pytest
import torch

import paper_2509_15763_amd as u
from paper_2509_15763_amd import synth
from _parity import TOL_GRAD_BF16, TOL_LSE_BF16, max_abs, oracle_fwd_bwd, out_ok, rel_l2, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [1, 2, 3, 4, 7, 8])
@pytest.mark.parametrize("L", [1, 31, 33, 129, 320])
def test_group_sizes(G, L):
    B, Hkv, D, r, W = 1, 2, 64, 3, 40
    q, k, v, do = synth.attn_inputs(B, G * Hkv, Hkv, L, D, seed=L + G)
    qd, kd, vd, dod = (t.cuda() for t in (q, k, v, do))
    out, lse = u.attn_fwd(qd, kd, vd, r, W)
    got = u.attn_bwd(qd, kd, vd, out, lse, dod, r, W)
    o, l, *want = oracle_fwd_bwd(q, k, v, do, r, W)
    assert out_ok(to_np(out), o) and max_abs(to_np(lse), l) <= TOL_LSE_BF16
    for a, b in zip(got, want):
        # a single token has dS = P (dP - delta) = 0 up to the rounding of the bf16 out in delta: absolute bound
        assert rel_l2(to_np(a), b) <= TOL_GRAD_BF16 if L > 4 else max_abs(to_np(a), b) <= 2e-2


@pytest.mark.parametrize("C", [3072, 4096, 4097])  # 768 workgroups: three per CU; 1024 and more: two per CU
def test_prefill_chunk_at_the_occupancy_rule(C):
    L, p0, r, W = 12288, 6144, 4, 256
    q, k, v, _ = (t.cuda() for t in synth.attn_inputs(1, 32, 8, L, 128, seed=C))
    out, lse = u.attn_fwd(q, k, v, r, W)
    cache = u.KVCache(1, 8, L, 128, r)
    cache.update(k[:, :, :p0 + C], v[:, :, :p0 + C], u.unigist_window_start(p0, r, W))
    o, l = u.prefill_chunk(q[:, :, p0:p0 + C].contiguous(), cache, r, W, p0)
    assert out_ok(to_np(o), to_np(out[:, :, p0:p0 + C]))
    assert max_abs(to_np(l), to_np(lse[:, :, p0:p0 + C])) <= TOL_LSE_BF16
