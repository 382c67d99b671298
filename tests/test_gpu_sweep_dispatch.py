"""The sweep's forms give the same bits (run with -m gpu), the form that each side takes read off the rule itself: heads by themselves and
among so many that the general form runs, and packed batches of few, more and many heads, where the rule counts the longest sequence's chunks."""
import os
import subprocess

import pytest

pytestmark = pytest.mark.gpu
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_16381_amd", "csrc")
SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include "sweep_form.h"
int main(int, char** v) { printf("%d", path::sweep_form(atoi(v[1]), atoi(v[2]), atoi(v[3]), atoi(v[4]) != 0)); }
"""


@pytest.fixture(scope="module")
def form(tmp_path_factory):
    d = tmp_path_factory.mktemp("form")
    (d / "form.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", f"-I{CSRC}", str(d / "form.cpp"), "-o", str(d / "form")], check=True)
    return lambda n, nc, heads, ring: int(subprocess.run([str(d / "form"), str(n), str(nc), str(heads), str(int(ring))], check=True, capture_output=True, text=True).stdout)


def _inputs(shape, d, seed):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rn = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    x = [rn(*shape, d).bfloat16() for _ in range(3)] + [torch.nn.functional.normalize(rn(*shape, d), dim=-1).bfloat16(), (2 * torch.sigmoid(rn(*shape))).bfloat16()]
    return x, torch.nn.functional.logsigmoid(rn(*shape) + 2).bfloat16()


def _workspace(nbytes):
    import torch
    return torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("gates", [False, True])
@pytest.mark.parametrize("d,L,few,many", [(64, 2113, 2, 48), (128, 3300, 7, 32), (128, 1024, 16, 72), (64, 700, 32, 96)])
def test_few_and_general(form, d, L, few, many, gates):
    import torch
    import paper_2505_16381_amd as pa
    chunks = -(-L // 64)
    assert form(chunks, chunks, few, False) in (1, 2) and form(chunks, chunks, many, False) == 0
    x, log_f = _inputs((1, many, L), d, L + d)
    out = []
    for H in (few, many):
        a, f = [t[:, :H].contiguous() for t in x], log_f[:, :H].contiguous() if gates else None
        o, lse = pa.path_attn_train_fwd(*a, _workspace(pa.path_attn_workspace_bytes(1, H, L, d, pa.PATH_BF16, True)), log_f=f, scale=d ** -0.5)
        out.append([o[:, :few], lse[:, :few]])
    for p, q in zip(*out):
        assert torch.isfinite(p).all() and torch.equal(p, q)


@pytest.mark.parametrize("gates", [False, True])
@pytest.mark.parametrize("d,lens", [(128, [2113, 64, 700, 1]), (64, [575, 2113, 130, 64])])
def test_packed(form, d, lens, gates):
    import torch
    import paper_2505_16381_amd as pa
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    chunks, counts = -(-max(lens) // 64), (2, 6, 16)
    assert [form(chunks, chunks, len(lens) * H, False) for H in counts] == [1, 2, 0]
    x, log_f = _inputs((cu[-1], counts[-1]), d, d)
    do = _inputs((cu[-1], counts[-1]), d, d + 1)[0][0]
    out = []
    for H in counts:
        a, f, g = [t[:, :H].contiguous() for t in x], log_f[:, :H].contiguous() if gates else None, do[:, :H].contiguous()
        o, lse = pa.path_attn_varlen_fwd(*a, cu, log_f=f, workspace=_workspace(pa.path_attn_varlen_workspace_bytes(cu, H, d, pa.PATH_BF16, False)))
        grads = pa.path_attn_varlen_bwd(*a, o, lse, g, cu, log_f=f, workspace=_workspace(pa.path_attn_varlen_workspace_bytes(cu, H, d, pa.PATH_BF16, True)))
        out.append([t[:, :2] for t in (o, lse, *grads[:5])])
    for other in out[1:]:
        for p, q in zip(out[0], other):
            assert torch.isfinite(p).all() and torch.equal(p, q)
