"""The sweep with waves of its own for the tile copies, which few workgroups take (16-bit operands; run with -m gpu): heads by
themselves have the bits they have among so many that the other form runs, plain and gated, forward and training pair, at
lengths around a chunk, a tile and a super-block."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gates", [False, True])
@pytest.mark.parametrize("d,L,few,many", [(128, 1, 1, 300), (64, 64, 3, 260), (128, 65, 2, 260), (128, 129, 5, 260), (64, 1024, 3, 40),
                                          (128, 1025, 4, 40), (128, 1100, 1, 32), (64, 2113, 2, 24), (128, 3300, 7, 24)])
def test_heads_by_themselves_and_among_many(d, L, few, many, gates):
    import torch
    import paper_2505_16381_amd as pa
    gen = torch.Generator(device="cuda").manual_seed(L + d)
    rn = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    x = [rn(1, many, L, d).bfloat16() for _ in range(3)] + [torch.nn.functional.normalize(rn(1, many, L, d), dim=-1).bfloat16(),
                                                            (2 * torch.sigmoid(rn(1, many, L))).bfloat16()]
    log_f = torch.nn.functional.logsigmoid(rn(1, many, L) + 2).bfloat16() if gates else None
    do = rn(1, many, L, d).bfloat16()
    tiles = -(-L // 128)
    assert few < 8 and many * tiles > 256 >= few * (tiles + 7)          # both forms (fewer than eight heads are dealt out to all XCDs)

    def run(sel):
        a, f, g = [t[:, sel].contiguous() for t in x], None if log_f is None else log_f[:, sel].contiguous(), do[:, sel].contiguous()
        H = a[0].shape[1]
        nan = lambda bwd: torch.full((pa.path_attn_workspace_bytes(1, H, L, d, pa.PATH_BF16, bwd),), 255, dtype=torch.uint8, device="cuda")
        out = list(pa.path_attn_fwd_layout(*a, pa.PATH_LAYOUT_BHLD, log_f=f, workspace=nan(False)))
        ws = nan(True)
        o, lse = pa.path_attn_train_fwd(*a, ws, log_f=f, scale=d ** -0.5)
        grads = pa.path_attn_train_bwd(*a, o, lse, g, ws, log_f=f, scale=d ** -0.5)
        return out + [o, lse] + list(grads[:5])

    for p, q in zip(run(slice(many - few, many)), run(slice(0, many))):
        assert torch.isfinite(p).all() and torch.equal(p, q[:, many - few:])


@pytest.mark.parametrize("gates", [False, True])
@pytest.mark.parametrize("d,L,few,many", [(128, 64, 1, 260), (64, 192, 3, 136), (128, 1088, 2, 32), (64, 2112, 4, 24)])
def test_ring_of_heads_by_themselves_and_among_many(d, L, few, many, gates):
    """Own segment and one hop (over a segment of another length), likewise."""
    import torch
    import paper_2505_16381_amd as pa
    gen = torch.Generator(device="cuda").manual_seed(7 * L + d)
    rn = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    Lk = L + 64

    def segment(n):
        return [rn(1, many, n, d).bfloat16() for _ in range(3)] + [torch.nn.functional.normalize(rn(1, many, n, d), dim=-1).bfloat16(),
                (2 * torch.sigmoid(rn(1, many, n))).bfloat16(), torch.nn.functional.logsigmoid(rn(1, many, n) + 2).bfloat16()]

    own, earlier = segment(L), segment(Lk)
    tiles = -(-L // 128)
    assert few < 8 and many * tiles > 256 >= few * (tiles + 7)

    def run(sel):
        H = len(range(many)[sel])
        nan = lambda n: torch.full((n,), 255, dtype=torch.uint8, device="cuda")
        ws = [nan(pa.path_attn_workspace_bytes(1, H, n, d, pa.PATH_BF16, False)) for n in (L, Lk)]
        st = [nan(pa.path_attn_ring_state_bytes(1, H, n, d)) for n in (L, Lk)]
        for i, seg in enumerate((own, earlier)):
            a = [t[:, sel].contiguous() for t in seg]
            pa.path_attn_ring_local(*a[:5], st[i], ws[i], log_f=a[5] if gates else None, scale=d ** -0.5)
        pa.path_attn_ring_hop(st[0], 1, H, L, ws[1], Lk, d, pa.PATH_BF16, with_gates=gates, scale=d ** -0.5)
        o, lse = torch.empty(1, H, L, d, dtype=torch.bfloat16, device="cuda"), torch.empty(1, H, L, device="cuda")
        pa.path_attn_ring_finish(st[0], o, lse, gates_workspace=ws[0] if gates else None)
        return o, lse

    for p, q in zip(run(slice(many - few, many)), run(slice(0, many))):
        assert torch.isfinite(p).all() and torch.equal(p, q[:, many - few:])
