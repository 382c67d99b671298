"""The fp32 far key sums at d = 64 number their workgroups over all heads of an XCD (run with -m gpu): with one, two and more
workgroups per CU, head counts that are no multiple of eight and packed sequences, the gradients are the bits of the backward
that passes over the heads one by one."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,L", [(5, 2113), (17, 1100), (33, 2113), (32, 2113), (20, 3137)])
def test_all_heads_at_once_and_one_by_one(H, L):
    import torch
    import paper_2505_16381_amd as pa
    d = 64
    gen = torch.Generator(device="cuda").manual_seed(H)
    rn = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    q, k, v, do = (rn(1, H, L, d) for _ in range(4))
    w, beta = torch.nn.functional.normalize(rn(1, H, L, d), dim=-1), 2 * torch.sigmoid(rn(1, H, L))
    o, lse = pa.path_attn_fwd(q, k, v, w, beta)
    grads = []
    for heads in (H, 1):
        ws = torch.full((pa.path_attn_bwd_workspace_bytes_for_heads(1, H, L, d, pa.PATH_F32, heads),), 255, dtype=torch.uint8, device="cuda")      # NaNs
        grads.append(pa.path_attn_bwd(q, k, v, w, beta, o, lse, do, workspace=ws))
    for a, b in zip(*grads):
        assert torch.isfinite(a).all() and torch.equal(a, b)


def test_packed_sequences_and_each_by_itself():
    import torch
    import paper_2505_16381_amd as pa
    d, H, lens = 64, 3, [1100, 64, 2113, 1025, 1, 1500]
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    gen = torch.Generator(device="cuda").manual_seed(7)
    rn = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    T = cu[-1]
    q, k, v, do = (rn(T, H, d) for _ in range(4))
    w, beta = torch.nn.functional.normalize(rn(T, H, d), dim=-1), 2 * torch.sigmoid(rn(T, H))
    o, lse = pa.path_attn_varlen_fwd(q, k, v, w, beta, cu)
    grads = pa.path_attn_varlen_bwd(q, k, v, w, beta, o, lse, do, cu)
    for a, b in zip(cu, cu[1:]):
        s = [t[a:b].unsqueeze(0).contiguous() for t in (q, k, v, w, beta)]
        so, sl = pa.path_attn_fwd_layout(*s, pa.PATH_LAYOUT_BLHD)
        assert torch.equal(so[0], o[a:b]) and torch.equal(sl[0], lse[a:b])
        for g, x in zip(pa.path_attn_bwd_layout(*s, so, sl, do[a:b].unsqueeze(0).contiguous(), pa.PATH_LAYOUT_BLHD), grads):
            assert torch.equal(g[0], x[a:b])
