"""GPU parity of the training pair in a workspace full of NaNs (run with -m gpu).

A training step leaves parts of its workspace unwritten -- the second-level tiles of a head's last super-block and
everything its adjoint would put there -- and no kernel may read them.  Lengths around the edges of a super-block
(1024 tokens; one, two, three, four query chunks right of the first), dense and packed; the bars are those of the other backward tests (2e-2 bf16, 1e-4 fp32, of the
tensor's maximum), which a single NaN fails.
"""
import numpy as np
import pytest

from paper_2505_16381_amd import synth_inputs as si

pytestmark = pytest.mark.gpu
TOL = {"fp32": 1e-4, "bf16": 2e-2}
NAMES = ("dq", "dk", "dv", "dw", "dbeta")


@pytest.fixture(scope="module")
def gpu():
    import torch
    import paper_2505_16381_amd as pa
    assert torch.cuda.is_available()
    pa.load_library()
    return torch, pa


def _nan_workspace(torch, nbytes):
    return torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")      # 0xFF..: NaN in every float type


def _compare(ref, got, dtype, tag):
    for n, r, g in zip(NAMES, ref, got):
        g = g.float().cpu().numpy().astype(np.float64)
        e = np.abs(g - r).max() / max(np.abs(r).max(), 1e-2)
        print(f"[{tag}] {n} {e:.2e}", flush=True)
        assert np.isfinite(g).all() and e <= TOL[dtype], (tag, n, e)


@pytest.mark.parametrize("dtype,L,d", [("bf16", 1024, 128), ("bf16", 1025, 64), ("bf16", 1089, 128), ("bf16", 1153, 64),
                                       ("bf16", 1217, 128), ("bf16", 2048, 128), ("bf16", 2111, 64),
                                       ("fp32", 1024, 64), ("fp32", 1089, 128)])
def test_training_pair(gpu, oracle, dtype, L, d):
    torch, pa = gpu
    scale = d ** -0.5
    x = si.make_inputs(1, 2, L, d, dtype, 3100 + L + d, 0.0, with_do=True)
    td, dt = (torch.float32, pa.PATH_F32) if dtype == "fp32" else (torch.bfloat16, pa.PATH_BF16)
    t = {n: torch.from_numpy(a).to("cuda").to(td).contiguous() for n, a in x.items()}
    ws = _nan_workspace(torch, pa.path_attn_workspace_bytes(1, 2, L, d, dt, True))
    o, lse = pa.path_attn_train_fwd(t["q"], t["k"], t["v"], t["w"], t["beta"], ws, scale=scale)
    grads = pa.path_attn_train_bwd(t["q"], t["k"], t["v"], t["w"], t["beta"], o, lse, t["dO"], ws, scale=scale)
    torch.cuda.synchronize()
    _compare(oracle.bwd(x["q"], x["k"], x["v"], x["w"], x["beta"], x["dO"], scale), grads, dtype, f"pair {dtype} L={L} d={d}")


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("fp32", 64)])
def test_packed_sequences(gpu, oracle, dtype, d):
    """Sequences of one, exactly one, two and (ragged) three super-blocks in one batch: every head its own last one."""
    torch, pa = gpu
    H, scale = 2, d ** -0.5
    lens = [700, 1024, 2048, 65, 2100]
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    x = si.make_inputs(1, H, cu[-1], d, dtype, 3200 + d, 0.0, with_do=True)
    td, dt = (torch.float32, pa.PATH_F32) if dtype == "fp32" else (torch.bfloat16, pa.PATH_BF16)
    t = {n: torch.from_numpy(np.ascontiguousarray(np.moveaxis(a[0], 0, 1))).to("cuda").to(td).contiguous() for n, a in x.items()}   # [T,H,(d)]
    ws = _nan_workspace(torch, pa.path_attn_varlen_workspace_bytes(cu, H, d, dt, True))
    o, lse = pa.path_attn_varlen_fwd(t["q"], t["k"], t["v"], t["w"], t["beta"], cu, scale=scale, workspace=ws)
    ws.fill_(255)
    grads = pa.path_attn_varlen_bwd(t["q"], t["k"], t["v"], t["w"], t["beta"], o, lse, t["dO"], cu, scale=scale, workspace=ws)
    torch.cuda.synchronize()
    for a, b in zip(cu, cu[1:]):
        s = {n: np.ascontiguousarray(v[:, :, a:b]) for n, v in x.items()}
        ref = oracle.bwd(s["q"], s["k"], s["v"], s["w"], s["beta"], s["dO"], scale)
        _compare(ref, [np_to(g, a, b) for g in grads], dtype, f"packed {dtype} d={d} L={b - a}")


def np_to(g, a, b):
    """Tokens a .. b-1 of a packed gradient [T,H,...] as [1,H,L,...]."""
    return g[a:b].movedim(0, 1)[None]
