"""A decoding step whose output takes the place of one of its inputs (run with -m gpu): with o over q, k or v the step gives
the bits of the step with an output of its own, unsplit and split, for heads of one and of two waves."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", ["q", "k", "v"])
@pytest.mark.parametrize("d,B,H,n", [(128, 6, 42, 0), (128, 6, 42, 60), (128, 6, 42, 500), (128, 6, 42, 1089), (64, 16, 31, 1100)])
def test_output_over_an_input(d, B, H, n, over):
    import torch
    import paper_2505_16381_amd as pa
    gen = torch.Generator().manual_seed(n + d)
    rn = lambda *s: torch.randn(*s, generator=gen).bfloat16().cuda()
    x = dict(q=rn(B, H, d), k=rn(B, H, d), v=rn(B, H, d))
    w = torch.nn.functional.normalize(rn(B, H, d), dim=-1)
    beta = (2 * torch.rand(B, H, generator=gen)).bfloat16().cuda()
    kc, vc = rn(B, H, n + 1, d), rn(B, H, n + 1, d)

    def step(o, **x):
        k2, v2, lse = kc.clone(), vc.clone(), torch.empty(B, H, device="cuda")
        pa.path_decode_step_static(x["q"], x["k"], x["v"], w, beta, k2, v2, n, d ** -0.5, o, lse)
        return o, lse, k2, v2

    want = step(torch.empty_like(x["q"]), **x)
    own = {m: t.clone() for m, t in x.items()}
    for a, b in zip(step(own[over], **own), want):
        assert torch.equal(a, b)
