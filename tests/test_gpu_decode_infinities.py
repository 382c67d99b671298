"""An infinite value in the cache makes its own component of a decoding step's output infinite and leaves the others alone
(run with -m gpu): at cache lengths that are not whole steps of a wave and with numbers of splits that are not whole batches
of the merge, where positions and splits past the end are stood in for by the last one with weight zero."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,n", [("bf16", 128, 1), ("bf16", 128, 33), ("bf16", 64, 129), ("bf16", 128, 500), ("bf16", 128, 1089),
                                       ("bf16", 64, 3001), ("fp32", 64, 7), ("fp32", 128, 250), ("fp32", 128, 1089)])
def test_infinite_values_stay_in_their_component(dtype, d, n):
    import torch
    import paper_2505_16381_amd as pa
    td = torch.float32 if dtype == "fp32" else torch.bfloat16
    gen = torch.Generator().manual_seed(n + d)
    rn = lambda *s: torch.randn(*s, generator=gen)
    B, H, Lmax = 1, 2, n + 3
    q, k, v = (rn(B, H, d).to(td).cuda() for _ in range(3))
    w = torch.nn.functional.normalize(rn(B, H, d), dim=-1).to(td).cuda()
    beta = (2 * torch.rand(B, H, generator=gen)).to(td).cuda()
    kc, vc = rn(B, H, Lmax, d).to(td).cuda(), rn(B, H, Lmax, d).to(td).cuda()
    inf = vc.clone()
    rows = {5: n - 1, 9: n // 2, 11: 0}                     # component: row
    for c, r in rows.items():
        inf[:, :, r, c] = float("inf")
    want, want_l = pa.path_decode_step(q, k, v, w, beta, kc.clone(), vc.clone(), n, d ** -0.5)
    got, got_l = pa.path_decode_step(q, k, v, w, beta, kc.clone(), inf, n, d ** -0.5)
    assert torch.isfinite(want).all() and torch.equal(got_l, want_l)
    others = [c for c in range(d) if c not in rows]
    assert torch.equal(got[:, :, others], want[:, :, others])
    assert (got[:, :, list(rows)] == float("inf")).all(), got[:, :, list(rows)]
