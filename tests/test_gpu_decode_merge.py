"""Splits of a decoding step merged inside its one launch (run with -m gpu): step after step in one workspace -- through the
numbers of splits and waves that the rules give, as the cache grows and for other shapes in between -- has the bits of a step
in a workspace of its own, filled with NaNs, and so has every replay of a captured step."""
import pytest

pytestmark = pytest.mark.gpu


def _make(torch, d, BH, n, dtype, seed):
    td = torch.float32 if dtype == "fp32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rn = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    x = [rn(1, BH, d).to(td) for _ in range(3)] + [torch.nn.functional.normalize(rn(1, BH, d), dim=-1).to(td), torch.rand(1, BH, device="cuda", generator=gen).to(td)]
    return x, rn(1, BH, n + 8, d).to(td), rn(1, BH, n + 8, d).to(td)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_one_workspace_for_all_steps(dtype):
    import torch
    import paper_2505_16381_amd as pa
    shapes = [(128, 16, 400), (128, 16, 1100), (64, 3, 1500), (128, 1, 9000), (64, 40, 5000), (128, 64, 1030), (64, 1, 4100), (128, 16, 400), (64, 70, 700)]
    ws = torch.full((max(pa.path_decode_workspace_bytes(1, BH, d) for d, BH, _ in shapes),), 255, dtype=torch.uint8, device="cuda")
    for rep in range(2):
        for i, (d, BH, n) in enumerate(shapes):
            x, kc, vc = _make(torch, d, BH, n, dtype, 10 * rep + i)
            k2, v2 = kc.clone(), vc.clone()
            for step in range(3):
                o, lse = pa.path_decode_step(*x, kc, vc, n + step, d ** -0.5, workspace=ws)
                own = torch.full((pa.path_decode_workspace_bytes(1, BH, d),), 255, dtype=torch.uint8, device="cuda")
                o2, lse2 = pa.path_decode_step(*x, k2, v2, n + step, d ** -0.5, workspace=own)
                assert torch.isfinite(o).all() and torch.equal(o, o2) and torch.equal(lse, lse2) and torch.equal(kc, k2) and torch.equal(vc, v2)


@pytest.mark.parametrize("d,BH,n", [(128, 16, 500), (64, 3, 3000)])
def test_replays_of_a_captured_split_step(d, BH, n):
    import torch
    import paper_2505_16381_amd as pa
    x, kc, vc = _make(torch, d, BH, n, "bf16", 5)
    k2, v2 = kc.clone(), vc.clone()
    ws = torch.empty(pa.path_decode_workspace_bytes(1, BH, d), dtype=torch.uint8, device="cuda")
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        pa.path_decode_step(*x, kc.clone(), vc.clone(), n, d ** -0.5, workspace=ws)
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        o, lse = pa.path_decode_step(*x, kc, vc, n, d ** -0.5, workspace=ws)
    for i in range(6):
        x[0].copy_(torch.randn(x[0].shape, device="cuda"))
        g.replay()
        o2, lse2 = pa.path_decode_step(*x, k2, v2, n, d ** -0.5)
        torch.cuda.synchronize()
        assert torch.equal(o, o2) and torch.equal(lse, lse2) and torch.equal(kc, k2) and torch.equal(vc, v2)
