"""The chunk transform for 16-bit operands where its chunk is ragged (run with -m gpu): one head's results at lengths that leave
1 .. 63 tokens in the last chunk, on both sides of its 32x32 blocks, against the oracle; heads contiguous and interleaved give the same
bits; a workspace full of NaNs shows up if anything is read that was not written (the diagonal logits right of the diagonal are not)."""
import numpy as np
import pytest

from paper_2505_16381_amd import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [1, 31, 32, 33, 63, 64, 65, 97, 160])
def test_ragged_chunk(oracle, d, L):
    import torch
    import paper_2505_16381_amd as pa
    B, H, scale = 1, 2, d ** -0.5
    x = si.make_inputs(B, H, L, d, "bf16", 9000 + L + d, 0.0, with_do=True)
    dv = {n: torch.from_numpy(a).to("cuda").bfloat16().contiguous() for n, a in x.items()}
    nan = lambda bwd: torch.full((pa.path_attn_workspace_bytes(B, H, L, d, pa.PATH_BF16, bwd),), 255, dtype=torch.uint8, device="cuda")
    args = [dv[n] for n in ("q", "k", "v", "w", "beta")]
    o, lse = pa.path_attn_fwd(*args, scale=scale, workspace=nan(False))
    grads = pa.path_attn_bwd(*args, o, lse, dv["dO"], scale=scale, workspace=nan(True))
    # interleaved heads
    turn = lambda t: t.transpose(1, 2).contiguous()
    targs = [turn(a) for a in args]
    o2, lse2 = pa.path_attn_fwd_layout(*targs, pa.PATH_LAYOUT_BLHD, scale=scale, workspace=nan(False))
    grads2 = pa.path_attn_bwd_layout(*targs, o2, lse2, turn(dv["dO"]), pa.PATH_LAYOUT_BLHD, scale=scale, workspace=nan(True))
    torch.cuda.synchronize()
    for a, b in zip([o, lse, *grads], [o2, lse2, *grads2]):
        assert torch.equal(a, turn(b))
    o_ref, lse_ref = oracle.fwd(x["q"], x["k"], x["v"], x["w"], x["beta"], scale)
    assert np.abs(o.float().cpu().numpy() - o_ref).max() <= 2e-2 and np.abs(lse.cpu().numpy() - lse_ref).max() <= 1e-3
    ref = oracle.bwd(x["q"], x["k"], x["v"], x["w"], x["beta"], x["dO"], scale)
    for g, r in zip(grads, ref):
        assert np.abs(g.float().cpu().numpy() - r).max() / max(np.abs(r).max(), 1e-2) <= 2e-2
