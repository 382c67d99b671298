"""Near key-side sums inside the chunk-transform adjoint, 16-bit operands (run with -m gpu): key chunks with no, one, some and
all fifteen query chunks to the right in their super-block, with and without queries beyond it, head counts that leave (super-block,
head) pairs over for the XCDs; whole heads against the oracle, and all heads at once against one by one, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,L,d", [(1, 64, 64), (1, 65, 128), (3, 129, 64), (5, 1024, 128), (9, 1025, 128), (9, 1100, 64),
                                   (3, 1984, 64), (2, 2113, 128)])
def test_gradients(H, L, d):
    import torch
    import paper_2505_16381_amd as pa
    from paper_2505_16381_amd import synth_inputs as si
    from oracle import path_oracle
    scale = d ** -0.5
    x = si.make_inputs(1, H, L, d, "bf16", 77 + L, 0.0, with_do=True)
    dev = {n: torch.from_numpy(a).to("cuda").to(torch.bfloat16).contiguous() for n, a in x.items()}
    args = [dev[n] for n in ("q", "k", "v", "w", "beta")]
    o, lse = pa.path_attn_fwd(*args, scale=scale)
    grads = []
    for heads in (H, 1):
        ws = torch.full((pa.path_attn_bwd_workspace_bytes_for_heads(1, H, L, d, pa.PATH_BF16, heads),), 255, dtype=torch.uint8, device="cuda")      # NaNs
        grads.append(pa.path_attn_bwd(*args, o, lse, dev["dO"], scale=scale, workspace=ws))
    for a, b in zip(*grads):
        assert torch.equal(a, b)
    sel = slice(H - 1, H)                        # the last head: its pairs are dealt last
    ref = path_oracle.bwd(*[np.ascontiguousarray(x[n][:, sel]) for n in ("q", "k", "v", "w", "beta", "dO")], scale)
    for g, r in zip(grads[0], ref):              # the bar of the other backward tests: 2e-2 of the tensor's maximum (bf16 rounds it to 2^-9)
        assert np.abs(g[:, sel].float().cpu().numpy() - r).max() <= 2e-2 * max(np.abs(r).max(), 1e-2)
