"""The fused chunk-transform adjoint with fp32 operands at d = 64 (run with -m gpu): lengths at the edges of a chunk and with one
chunk beyond a super-block, both layouts, plain and gated, every gradient against the oracle; the bar is that of the other fp32
backward tests, 1e-4 of the tensor's maximum."""
import numpy as np
import pytest

from paper_2505_16381_amd import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["BHLD", "BLHD"])
@pytest.mark.parametrize("gates", [False, True])
@pytest.mark.parametrize("L", [1, 31, 64, 65, 130, 1060])
def test_gradients(L, gates, layout):
    import torch
    import paper_2505_16381_amd as pa
    from oracle import path_oracle
    d, H = 64, 3
    x = si.make_inputs(1, H, L, d, "fp32", 900 + L, 0.0, with_do=True)
    logf = np.log(1.0 / (1.0 + np.exp(-(np.random.default_rng(L).standard_normal((1, H, L)) + 2.0)))).astype(np.float32) if gates else None
    t = (lambda a: torch.from_numpy(np.ascontiguousarray(a if layout == "BHLD" else a.swapaxes(1, 2))).cuda())
    args, f, do = [t(x[n]) for n in ("q", "k", "v", "w", "beta")], t(logf) if gates else None, t(x["dO"])
    lay = pa.PATH_LAYOUT_BHLD if layout == "BHLD" else pa.PATH_LAYOUT_BLHD
    o, lse = pa.path_attn_fwd_layout(*args, lay, log_f=f)
    ws = torch.full((pa.path_attn_workspace_bytes(1, H, L, d, pa.PATH_F32, True),), 255, dtype=torch.uint8, device="cuda")      # NaNs
    got = pa.path_attn_bwd_layout(*args, o, lse, do, lay, log_f=f, workspace=ws)
    ref = path_oracle.bwd(x["q"], x["k"], x["v"], x["w"], x["beta"], x["dO"], d ** -0.5, logf=logf)
    for g, r in zip(got, ref):
        g = g.double().cpu().numpy()
        g = g if layout == "BHLD" else g.swapaxes(1, 2)
        assert np.abs(g - r).max() <= 1e-4 * max(np.abs(r).max(), 1e-2)
