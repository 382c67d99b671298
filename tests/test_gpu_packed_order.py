"""Packed batches on both sides of the rule that turns the heads by one per chunk (run with -m gpu): head counts below, at and
beside a multiple of eight, few and many chunks, the heads in one and in several passes of the backward; each sequence has the
bits it has by itself."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,H,lens,passes", [
    ("bf16", 128, 2, [292, 200, 100, 56], 1),                    # 5 chunks x 1: not turned
    ("bf16", 64, 2, [1100, 900, 65, 700, 500, 456, 1, 640], 1),  # 18 x 2: turned
    ("bf16", 128, 3, [2049, 64, 130], 1),                        # 33 x 2, nine heads
    ("bf16", 64, 3, [2049, 64, 130], 2),                         # ... in passes of fewer heads
    ("bf16", 64, 8, [700, 100, 1030], 1),                        # eight heads each: never turned
    ("fp32", 64, 4, [1025, 129, 640, 320, 64], 1)])
def test_sequences_in_a_batch_and_by_themselves(dtype, d, H, lens, passes):
    import torch
    import paper_2505_16381_amd as pa
    td = torch.float32 if dtype == "fp32" else torch.bfloat16
    dt = pa.PATH_F32 if dtype == "fp32" else pa.PATH_BF16
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    gen = torch.Generator(device="cuda").manual_seed(d + H)
    rn = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    q, k, v, do = (rn(cu[-1], H, d).to(td) for _ in range(4))
    w, beta = torch.nn.functional.normalize(rn(cu[-1], H, d), dim=-1).to(td), (2 * torch.sigmoid(rn(cu[-1], H))).to(td)
    nan = lambda nbytes: torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
    o, lse = pa.path_attn_varlen_fwd(q, k, v, w, beta, cu, workspace=nan(pa.path_attn_varlen_workspace_bytes(cu, H, d, dt, False)))
    nbytes = pa.path_attn_varlen_workspace_bytes(cu, H, d, dt, True)
    if passes > 1:
        heads = -(-len(lens) * H // passes)
        nbytes = 256 + pa.path_attn_bwd_workspace_bytes_for_heads(len(lens), H, max(lens), d, dt, heads)
    grads = pa.path_attn_varlen_bwd(q, k, v, w, beta, o, lse, do, cu, workspace=nan(nbytes))
    for a, b in zip(cu, cu[1:]):
        s = [t[a:b].unsqueeze(0).contiguous() for t in (q, k, v, w, beta)]
        so, sl = pa.path_attn_fwd_layout(*s, pa.PATH_LAYOUT_BLHD)
        assert torch.equal(so[0], o[a:b]) and torch.equal(sl[0], lse[a:b])
        for g, x in zip(pa.path_attn_bwd_layout(*s, so, sl, do[a:b].unsqueeze(0).contiguous(), pa.PATH_LAYOUT_BLHD), grads):
            assert torch.equal(g[0], x[a:b])
