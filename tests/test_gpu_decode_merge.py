"""Merge of the splits of a decoding step (run with -m gpu): step after step in one workspace -- through the
numbers of splits and waves that the rules give, as the cache grows and for other shapes in between -- has the bits of a step
in a workspace of its own, filled with NaNs, and so has every replay of a captured step, whatever its workspace holds."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

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


@pytest.mark.parametrize("gates", [False, True])
def test_replays_between_eager_steps_of_other_shapes(gates):
    """One workspace for a captured step and for eager ones before, between and after its replays."""
    import torch
    import paper_2505_16381_amd as pa
    d, BH, n = 128, 16, 1500
    others = [(128, 16, 700), (64, 3, 1500), (128, 1, 9000), (64, 40, 5000)]
    ws = torch.full((max(pa.path_decode_workspace_bytes(1, b, e) for e, b, _ in others + [(d, BH, n)]),), 255, dtype=torch.uint8, device="cuda")

    def caches(d, BH, n, seed):
        x, kc, vc = _make(torch, d, BH, n, "bf16", seed)
        gen = torch.Generator(device="cuda").manual_seed(seed)
        lf = lambda *s: torch.nn.functional.logsigmoid(torch.randn(*s, device="cuda", generator=gen) + 2)
        return x, lf(1, BH).bfloat16(), [kc, vc] + ([torch.cumsum(lf(1, BH, n + 8), -1)] if gates else [])

    def step(x, lf, c, n, d, workspace):
        if gates:
            return pa.path_decode_step_fox(*x, lf, *c, n, d ** -0.5, workspace=workspace)
        return pa.path_decode_step(*x, *c, n, d ** -0.5, workspace=workspace)

    x, lf, c = caches(d, BH, n, 5)
    c2 = [t.clone() for t in c]
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        step(x, lf, [t.clone() for t in c], n, d, ws)
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        o, lse = step(x, lf, c, n, d, ws)
    for i in range(2 * len(others)):
        e, b, m = others[i % len(others)]
        y, f, k = caches(e, b, m, i)
        k2 = [t.clone() for t in k]
        for a, r in zip((*step(y, f, k, m, e, ws), *k), (*step(y, f, k2, m, e, None), *k2)):
            assert torch.equal(a, r)
        g.replay()
        for a, r in zip((o, lse, *c), (*step(x, lf, c2, n, d, None), *c2)):
            assert torch.equal(a, r), i


SCRIPT = """
import sys
sys.path.insert(0, sys.argv[1])
import torch
import paper_2505_16381_amd as pa
BH, n, d = 64, 4000, 128
gen = torch.Generator(device="cuda").manual_seed(1)
rn = lambda *s: torch.randn(*s, device="cuda", generator=gen)
x = [rn(1, BH, d).bfloat16() for _ in range(3)] + [torch.nn.functional.normalize(rn(1, BH, d), dim=-1).bfloat16(), torch.rand(1, BH, device="cuda", generator=gen).bfloat16()]
kc, vc = rn(1, BH, n + 8, d).bfloat16(), rn(1, BH, n + 8, d).bfloat16()
k2, v2 = kc.clone(), vc.clone()
ws = torch.zeros(pa.path_decode_workspace_bytes(1, BH, d) // 8, dtype=torch.int64, device="cuda")
st = torch.cuda.Stream()
with torch.cuda.stream(st):
    pa.path_decode_step(*x, kc.clone(), vc.clone(), n, d ** -0.5, workspace=ws.view(torch.uint8))
st.synchronize()
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g, stream=st):
    o, lse = pa.path_decode_step(*x, kc, vc, n, d ** -0.5, workspace=ws.view(torch.uint8))
for call in range(1, 5):
    mark = call * 0x9E3779B97F4A7C15 % 2 ** 64
    ws.fill_(mark - 2 ** 64 if mark >= 2 ** 63 else mark)              # (also as the maxima and sums of records)
    g.replay()
    want = pa.path_decode_step(*x, k2, v2, n, d ** -0.5)
    torch.cuda.synchronize()
    print(call, *[bool(torch.equal(a, b)) for a, b in zip((o, lse, kc, vc), (*want, k2, v2))], flush=True)
"""


def test_marks_of_earlier_calls_in_the_workspace_of_a_replay():
    """The workspace is filled with the marks that the first calls of a process put on finished records, the captured call's
    among them, as a replay that did not end properly could leave them: in a process of its own, whose calls are counted."""
    r = subprocess.run([sys.executable, "-c", SCRIPT, ROOT], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    assert [l.split()[1:] for l in r.stdout.splitlines() if l[:1].isdigit()] == [["True"] * 4] * 4, r.stdout
