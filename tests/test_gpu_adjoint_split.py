"""The adjoint scan's two kernels for 16-bit operands (run with -m gpu): d = 128 takes the one split by kind of work from
nine chunks on.  The number of chunks is that of a batch's longest sequence, so a short sequence runs through one of them
alone and through the other beside a longer one: the same bits.  Lengths around the edges of that rule, of a workgroup
(four chunks) and of a super-block, with and without gates, are held against the oracle; bars as for the other backward
tests (2e-2 of the tensor's maximum, and of 1e-2 at least)."""
import numpy as np
import pytest

from paper_2505_16381_amd import synth_inputs as si

pytestmark = pytest.mark.gpu


def test_short_sequences_alone_and_beside_a_longer_one():
    import torch
    import paper_2505_16381_amd as pa
    H, d = 3, 128
    lens = [1, 64, 65, 200, 257, 449, 512, 577]
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    g = torch.Generator(device="cuda").manual_seed(11)
    q, k, v, w, do = (torch.randn((cu[-1], H, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(5))
    w = torch.nn.functional.normalize(w.float(), dim=-1).to(torch.bfloat16)
    beta = (torch.rand((cu[-1], H), generator=g, device="cuda") * 2).to(torch.bfloat16)

    def run(a, b, cu):
        x = [t[a:b].contiguous() for t in (q, k, v, w, beta)]
        ws = torch.full((pa.path_attn_varlen_workspace_bytes(cu, H, d, pa.PATH_BF16, True),), 255, dtype=torch.uint8, device="cuda")
        o, lse = pa.path_attn_varlen_fwd(*x, cu, workspace=ws)
        return pa.path_attn_varlen_bwd(*x, o, lse, do[a:b].contiguous(), cu, workspace=ws)

    together = run(0, cu[-1], cu)
    for a, b in list(zip(cu, cu[1:]))[:-1]:
        for name, x, y in zip(("dq", "dk", "dv", "dw", "dbeta"), run(a, b, [0, b - a]), together):
            assert bool(torch.isfinite(x).all()) and torch.equal(x, y[a:b]), (b - a, name)


@pytest.mark.parametrize("gates", [False, True])
@pytest.mark.parametrize("L", [512, 513, 577, 768, 1090])
def test_against_the_oracle(oracle, L, gates):
    import torch
    import paper_2505_16381_amd as pa
    H, d = 2, 128
    x = si.make_inputs(1, H, L, d, "bf16", 4100 + L, 0.0, with_do=True)
    t = {n: torch.from_numpy(a).to("cuda").to(torch.bfloat16).contiguous() for n, a in x.items()}
    args = [t[n] for n in ("q", "k", "v", "w", "beta")]
    ws = torch.full((pa.path_attn_workspace_bytes(1, H, L, d, pa.PATH_BF16, True),), 255, dtype=torch.uint8, device="cuda")
    logf = None
    if gates:
        lf = torch.nn.functional.logsigmoid(torch.randn((1, H, L), generator=torch.Generator().manual_seed(L)) + 3).to(torch.bfloat16)
        logf = lf.double().numpy()
        o, lse = pa.path_attn_fox_fwd(*args, lf.cuda(), workspace=ws)
        got = pa.path_attn_fox_bwd(*args, lf.cuda(), o, lse, t["dO"], workspace=ws)
    else:
        o, lse = pa.path_attn_fwd(*args, workspace=ws)
        got = pa.path_attn_bwd(*args, o, lse, t["dO"], workspace=ws)
    ref = oracle.bwd(x["q"], x["k"], x["v"], x["w"], x["beta"], x["dO"], d ** -0.5, logf=logf)
    for name, r, y in zip(("dq", "dk", "dv", "dw", "dbeta", "dlogf"), ref, got):
        y = y.double().cpu().numpy()
        e = np.abs(y - r).max() / max(np.abs(r).max(), 1e-2)
        print(f"[adjoint L={L} gates={gates}] {name} {e:.2e}", flush=True)
        assert np.isfinite(y).all() and e <= 2e-2, (name, e)
