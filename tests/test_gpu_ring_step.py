"""unigist_cache_ring_step: one launch appends a token per sequence and advances the positions in place.  More heads than
a workgroup has waves, inactive sequences, sequences that do not fit, against the rule of the ring layout spelled out."""
import pytest
import torch

import paper_2509_15763_amd as u

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hkv", [1, 3, 16, 17, 33])
@pytest.mark.parametrize("D", [8, 64, 128])
def test_step_against_the_layout(Hkv, D):
    B, r, W, cap = 4, 3, 10, 24
    gen = torch.Generator().manual_seed(Hkv * D)
    kc, vc = (torch.randn(B, Hkv, cap, D, generator=gen).bfloat16() for _ in range(2))
    kd, vd = kc.cuda(), vc.cuda()
    t = [-1, 9, 13, 62]  # empty; window just full; a gist leaves at 13 + 1 - 10 = 4 - 1; 10 + 16 rows: does not fit in 24
    td = torch.tensor(t, dtype=torch.int32).cuda()
    rows = torch.empty(B, dtype=torch.int32).cuda()
    for step, active in enumerate(([1, 1, 1, 1], None, [1, 0, 1, 1], None)):
        kn, vn = (torch.randn(B, Hkv, 1, D, generator=gen).bfloat16() for _ in range(2))
        act = None if active is None else torch.tensor(active, dtype=torch.int32).cuda()
        knd, vnd = kn.cuda(), vn.cuda()
        rc = u.unigist_cache_ring_step(kd.data_ptr(), vd.data_ptr(), knd.data_ptr(), vnd.data_ptr(), 1, td.data_ptr(),
                                       None if act is None else act.data_ptr(), cap, rows.data_ptr(), B, Hkv, D, r, W, 0,
                                       u.UNIGIST_WINDOW_SLIDING, u.UNIGIST_BF16, None)
        assert rc == 0
        torch.cuda.synchronize()
        want = []
        for b in range(B):
            a = 1 if active is None else active[b]
            n = u.unigist_cache_ring_rows(t[b] + a, r, W)
            if n > cap:
                want.append(-1)
                continue
            want.append(n)
            if not a:
                continue
            t[b] += 1
            out = t[b] - W  # the position that leaves the window: kept behind it if it is a gist
            for c, new in ((kc, kn), (vc, vn)):
                if out >= 0 and (out + 1) % (r + 1) == 0:
                    c[b, :, W + out // (r + 1)] = c[b, :, t[b] % W]
                c[b, :, t[b] % W] = new[b, :, 0]
        assert rows.tolist() == want and td.tolist() == t, step
        assert torch.equal(kd.cpu(), kc) and torch.equal(vd.cpu(), vc)
