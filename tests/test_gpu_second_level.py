"""The second-level transform's launch shapes and the key prefill of one super-block (run with -m gpu).

Many super-blocks run several workgroups per CU and few run one, with the same products in the same order, so a head's
results do not depend on how many heads run beside it: bit for bit.  The prefill is held against the decode oracle at
the edges of a chunk and of a super-block; bars as for the other prefill test (fp32 1e-4; bf16 the rounding of the
stored key, half a step of 2^-8 relative, and as much again for the 16-bit operands of the chain)."""
import numpy as np
import pytest

from paper_2505_16381_amd import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    import paper_2505_16381_amd as pa
    assert torch.cuda.is_available()
    pa.load_library()
    return torch, pa


@pytest.mark.parametrize("d,H,L", [(64, 257, 1089), (128, 257, 1089), (128, 129, 2111)])
def test_a_head_alone_and_among_many(gpu, d, H, L):
    torch, pa = gpu
    g = torch.Generator(device="cuda").manual_seed(5 + d + L)
    x = {n: torch.randn((1, H, L, d), generator=g, device="cuda").to(torch.bfloat16) for n in ("q", "k", "v", "w", "do")}
    x["w"] = torch.nn.functional.normalize(x["w"].float(), dim=-1).to(torch.bfloat16)
    x["beta"] = (torch.rand((1, H, L), generator=g, device="cuda") * 2).to(torch.bfloat16)

    def run(h0, h1):
        q, k, v, w, beta, do = (x[n][:, h0:h1].contiguous() for n in ("q", "k", "v", "w", "beta", "do"))
        ws = torch.empty(pa.path_attn_workspace_bytes(1, h1 - h0, L, d, pa.PATH_BF16, True), dtype=torch.uint8, device="cuda")
        o, lse = pa.path_attn_train_fwd(q, k, v, w, beta, ws)
        return (o, lse) + pa.path_attn_train_bwd(q, k, v, w, beta, o, lse, do, ws)

    many = run(0, H)
    for h in (0, H // 2, H - 1):
        for a, b in zip(run(h, h + 1), many):
            assert torch.equal(a[:, 0], b[:, h]), (d, H, L, h)


@pytest.mark.parametrize("dtype,d", [("fp32", 64), ("fp32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("L", [1, 63, 65, 960, 1024, 1025])
def test_prefill_at_the_edges(gpu, dtype, d, L):
    torch, pa = gpu
    from oracle import decode_oracle
    x = si.make_inputs(1, 2, L, d, dtype, 70 + L + d, 0.0)
    td = torch.float32 if dtype == "fp32" else torch.bfloat16
    dv = {n: torch.from_numpy(a).to("cuda").to(td).contiguous() for n, a in x.items()}
    nb = pa.path_attn_workspace_bytes(1, 2, L, d, pa.PATH_F32 if dtype == "fp32" else pa.PATH_BF16, False)
    ws = torch.full((nb,), 0xFF, dtype=torch.uint8, device="cuda")
    pa.path_attn_fwd_prep(dv["q"], dv["k"], dv["v"], dv["w"], dv["beta"], ws)
    kc = torch.full((1, 2, L + 3, d), 7.0, dtype=td, device="cuda")
    vc = torch.full((1, 2, L + 3, d), 7.0, dtype=td, device="cuda")
    pa.path_key_prefill(dv["v"], ws, kc, vc)
    want = decode_oracle.key_prefill(x["k"], x["w"], x["beta"])
    err = np.abs(kc[:, :, :L].float().cpu().numpy() - want).max()
    tol = 1e-4 if dtype == "fp32" else 2.0 ** -8 * np.abs(want).max() * 1.5
    print(f"[prefill {dtype} L={L} d={d}] max|dk|={err:.2e} (bar {tol:.2e})", flush=True)
    assert err <= tol
    assert torch.equal(vc[:, :, :L], dv["v"]) and bool((kc[:, :, L:] == 7).all()) and bool((vc[:, :, L:] == 7).all())
