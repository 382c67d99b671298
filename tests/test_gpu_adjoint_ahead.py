"""The adjoint scan at d = 64, 16-bit operands, whose workgroups bring the next chunk's tiles and the next block's state during a
step (run with -m gpu): lengths around a chunk, a workgroup (two chunks) and a super-block (sixteen), odd and even numbers of
chunks, with and without gates, in a workspace of NaN, against the oracle; bars as for the other backward tests (2e-2 of the
tensor's maximum, and of 1e-2 at least)."""
import numpy as np
import pytest

from paper_2505_16381_amd import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gates", [False, True])
@pytest.mark.parametrize("L", [1, 64, 65, 129, 1024, 1025, 1089, 2113])
def test_against_the_oracle(oracle, L, gates):
    import torch
    import paper_2505_16381_amd as pa
    H, d = 2, 64
    x = si.make_inputs(1, H, L, d, "bf16", 6200 + L, 0.0, with_do=True)
    t = {n: torch.from_numpy(a).to("cuda").to(torch.bfloat16).contiguous() for n, a in x.items()}
    args = [t[n] for n in ("q", "k", "v", "w", "beta")]
    ws = torch.full((pa.path_attn_workspace_bytes(1, H, L, d, pa.PATH_BF16, True),), 255, dtype=torch.uint8, device="cuda")
    logf = lf = None
    if gates:
        lf = torch.nn.functional.logsigmoid(torch.randn((1, H, L), generator=torch.Generator().manual_seed(L)) + 3).to(torch.bfloat16)
        logf, lf = lf.double().numpy(), lf.cuda()
    o, lse = pa.path_attn_train_fwd(*args, ws, log_f=lf, scale=d ** -0.5)
    got = pa.path_attn_train_bwd(*args, o, lse, t["dO"], ws, log_f=lf, scale=d ** -0.5)
    ref = oracle.bwd(x["q"], x["k"], x["v"], x["w"], x["beta"], x["dO"], d ** -0.5, logf=logf)
    for name, r, y in zip(("dq", "dk", "dv", "dw", "dbeta", "dlogf"), ref, got):
        y = y.double().cpu().numpy()
        e = np.abs(y - r).max() / max(np.abs(r).max(), 1e-2)
        print(f"[adjoint L={L} gates={gates}] {name} {e:.2e}", flush=True)
        assert np.isfinite(y).all() and e <= 2e-2
