"""dw and dbeta of the chunk-transform adjoint to the bit (run with -m gpu): the order in which a row of M o G is summed for dbeta, and how
beta M and its mirror image are rounded for dw, are fixed; recorded before the adjoint's tiles were turned, when M lay in LDS as 32-bit numbers."""
import hashlib

import pytest

from paper_2505_16381_amd import synth_inputs as si

pytestmark = pytest.mark.gpu

RECORDED = {        # (dtype, d, tokens): dw, dbeta
    ("bf16", 64, 1100): ("ac9aabfc857281b4", "5f9747aa64ade6e6"),
    ("bf16", 128, 1100): ("848d3c8ffbd3e238", "741b98e422c1d70b"),
    ("fp32", 64, 130): ("21523109588f51a7", "75df8e62204e7be8"),
    ("fp32", 64, 1100): ("36693b5ca53cb3a6", "7b52d0e61f939ad5"),
}


@pytest.mark.parametrize("dtype,d,L", sorted(RECORDED))
def test_as_recorded(dtype, d, L):
    import torch
    import paper_2505_16381_amd as pa
    x = si.make_inputs(1, 2, L, d, dtype, 300 + L, 0.0, with_do=True)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    t = {n: torch.from_numpy(a).to("cuda").to(td).contiguous() for n, a in x.items()}
    args = [t[n] for n in ("q", "k", "v", "w", "beta")]
    o, lse = pa.path_attn_fwd(*args, scale=d ** -0.5)
    grads = pa.path_attn_bwd(*args, o, lse, t["dO"], scale=d ** -0.5)
    digest = lambda g: hashlib.sha256(g.cpu().contiguous().view(torch.uint8).numpy().tobytes()).hexdigest()[:16]
    assert (digest(grads[3]), digest(grads[4])) == RECORDED[dtype, d, L]
