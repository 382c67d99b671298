"""The forms of the forward sweep -- one query chunk per workgroup, two, and the general one; which one runs is a matter of the number of
workgroups and of the chains' length -- give the same bits (run with -m gpu): heads by themselves and among as many as take another form, plain and
gated, forward, training pair and ring, with a chunk left over, whole super-blocks and short chains."""
import pytest

pytestmark = pytest.mark.gpu


def _inputs(H, L, d, td):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(3 * L + d)
    rn = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    x = [rn(1, H, L, d).to(td) for _ in range(3)] + [torch.nn.functional.normalize(rn(1, H, L, d), dim=-1).to(td), (2 * torch.sigmoid(rn(1, H, L))).to(td)]
    return x, torch.nn.functional.logsigmoid(rn(1, H, L) + 2).to(td)


def _workspace(nbytes):
    import torch
    return torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("gates", [False, True])
@pytest.mark.parametrize("dtype,d,L,counts", [
    ("bf16", 128, 2113, (3, 24, 64)),       # one chunk per workgroup, two (34 chunks), the general form
    ("bf16", 64, 2048, (9, 40, 96)),        # likewise, whole super-blocks
    ("bf16", 128, 190, (40, 120, 200)),     # three chunks: one, two (one left over), the general form
    ("bf16", 64, 575, (33, 56, 120)),       # nine chunks: one round, two rounds, the general form
    ("fp32", 64, 600, (4, 40, 60)),         # fp32: one round, two rounds, the general form
    ("fp32", 64, 1100, (2, 40)),
])
def test_forward_and_training_pair(dtype, d, L, counts, gates):
    import torch
    import paper_2505_16381_amd as pa
    td, dt = (torch.bfloat16, pa.PATH_BF16) if dtype == "bf16" else (torch.float32, pa.PATH_F32)
    x, log_f = _inputs(max(counts), L, d, td)
    few = min(counts)

    def run(H):
        a, f = [t[:, :H].contiguous() for t in x], log_f[:, :H].contiguous() if gates else None
        out = list(pa.path_attn_fwd_layout(*a, pa.PATH_LAYOUT_BHLD, log_f=f, workspace=_workspace(pa.path_attn_workspace_bytes(1, H, L, d, dt, False))))
        ws = _workspace(pa.path_attn_workspace_bytes(1, H, L, d, dt, True))
        o, lse = pa.path_attn_train_fwd(*a, ws, log_f=f, scale=d ** -0.5)
        grads = pa.path_attn_train_bwd(*a, o, lse, torch.ones_like(o), ws, log_f=f, scale=d ** -0.5)
        return [t[:, :few] for t in out + [o, lse] + list(grads[:5])]

    first = run(counts[0])
    for H in counts[1:]:
        for p, q in zip(first, run(H)):
            assert torch.isfinite(p).all() and torch.equal(p, q)


@pytest.mark.parametrize("gates", [False, True])
@pytest.mark.parametrize("d,Lq,Lk,counts", [(128, 3072, 3072, (3, 16, 40)),      # one chunk per workgroup, two (48 chunks), the general form
                                            (64, 192, 1088, (9, 120, 200)),      # a chunk left over, a product right at the hop's start
                                            (128, 65, 64, (8, 200))])
def test_ring(d, Lq, Lk, counts, gates):
    import torch
    import paper_2505_16381_amd as pa
    few = min(counts)
    own, earlier = _inputs(max(counts), Lq, d, torch.bfloat16), _inputs(max(counts), Lk, d, torch.bfloat16)

    def run(H):
        ws = [_workspace(pa.path_attn_workspace_bytes(1, H, n, d, pa.PATH_BF16, False)) for n in (Lq, Lk)]
        st = [_workspace(pa.path_attn_ring_state_bytes(1, H, n, d)) for n in (Lq, Lk)]
        for i, (x, f) in enumerate((own, earlier)):
            pa.path_attn_ring_local(*[t[:, :H].contiguous() for t in x], st[i], ws[i], log_f=f[:, :H].contiguous() if gates else None, scale=d ** -0.5)
        pa.path_attn_ring_hop(st[0], 1, H, Lq, ws[1], Lk, d, pa.PATH_BF16, with_gates=gates, scale=d ** -0.5)
        o, lse = torch.empty(1, H, Lq, d, dtype=torch.bfloat16, device="cuda"), torch.empty(1, H, Lq, device="cuda")
        pa.path_attn_ring_finish(st[0], o, lse, gates_workspace=ws[0] if gates else None)
        return [o[:, :few], lse[:, :few]]

    first = run(counts[0])
    for H in counts[1:]:
        for p, q in zip(first, run(H)):
            assert torch.isfinite(p).all() and torch.equal(p, q)
