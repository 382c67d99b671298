"""fp32 operands at d = 64 share 32 rows of the second level's matrix between two waves (run with -m gpu): keys in the cache
and forward rows at the edges of chunks and super-blocks, where a chain is one chunk, whole, or ragged, against the oracles."""
import numpy as np
import pytest

from paper_2505_16381_amd import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 64, 65, 129, 1024, 1025, 1089, 2113])
def test_keys_and_rows_against_the_oracles(L, oracle):
    import torch
    import paper_2505_16381_amd as pa
    from oracle import decode_oracle
    B, H, d = 1, 3, 64
    x = si.make_inputs(B, H, L, d, "fp32", 8100 + L, 0.0)
    t = {n: torch.from_numpy(a).cuda().contiguous() for n, a in x.items()}
    ws = torch.full((pa.path_attn_workspace_bytes(B, H, L, d, pa.PATH_F32, False),), 255, dtype=torch.uint8, device="cuda")     # NaNs
    o, lse = pa.path_attn_fwd(t["q"], t["k"], t["v"], t["w"], t["beta"], scale=d ** -0.5, workspace=ws)
    kc = torch.zeros(B, H, L + 1, d, device="cuda")
    vc = torch.zeros_like(kc)
    pa.path_key_prefill(t["v"], ws, kc, vc)
    f = lambda a: a.double().cpu().numpy()
    o_ref, l_ref = oracle.fwd(x["q"], x["k"], x["v"], x["w"], x["beta"], d ** -0.5)
    k_ref = decode_oracle.key_prefill(x["k"], x["w"], x["beta"])
    e = np.abs(f(o) - o_ref).max(), np.abs(f(lse) - l_ref).max(), np.abs(f(kc)[:, :, :L] - k_ref).max()
    print(f"[fp32 d=64 L={L}] max|do|={e[0]:.2e} max|dlse|={e[1]:.2e} max|dk|={e[2]:.2e}", flush=True)
    assert e[0] <= 1e-4 and e[1] <= 1e-3 and e[2] <= 1e-4        # the bars of the other fp32 tests
    assert torch.equal(vc[:, :, :L], t["v"]) and float(kc[:, :, L:].abs().max()) == 0.0
