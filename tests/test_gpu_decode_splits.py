"""GPU parity of one decoding step at the edges of its launch rules (run with -m gpu): cache lengths around a step of
four and of sixteen waves, around the largest head that one workgroup takes -- 64 KB of keys for few heads, 88 KB of fp32 ones, 88 KB
of bf16 ones for 64 heads, 128 KB for many --, around a multiple of the split length, with the largest number of splits, with
splits of four waves for many heads and with records that a second launch merges, from caches of random content, plain and
gated, against the decode oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gates", [False, True])
@pytest.mark.parametrize("dtype,d,B,H,n", [
    ("bf16", 128, 1, 3, 0), ("bf16", 64, 1, 2, 1), ("bf16", 128, 2, 2, 33), ("bf16", 64, 1, 3, 128), ("bf16", 64, 1, 3, 129),
    ("bf16", 128, 1, 2, 512), ("bf16", 128, 1, 2, 513), ("bf16", 64, 2, 2, 1024), ("bf16", 64, 2, 2, 1025), ("bf16", 128, 1, 2, 1089),
    ("bf16", 128, 1, 1, 8200), ("bf16", 64, 16, 65, 1100), ("fp32", 128, 1, 2, 129), ("fp32", 128, 1, 2, 256),
    ("fp32", 128, 1, 2, 257), ("fp32", 64, 1, 2, 513), ("fp32", 64, 1, 1, 5000), ("fp32", 128, 1, 1, 4100), ("fp32", 128, 1, 2, 8200),
    # one workgroup and the first length that is split
    ("bf16", 128, 1, 2, 129), ("bf16", 128, 1, 2, 256), ("bf16", 128, 1, 2, 257), ("bf16", 64, 1, 3, 512), ("bf16", 64, 1, 3, 513),
    ("bf16", 128, 4, 16, 352), ("bf16", 128, 4, 16, 353), ("bf16", 128, 7, 16, 512), ("bf16", 128, 7, 16, 513),
    ("fp32", 128, 1, 2, 176), ("fp32", 128, 1, 2, 177), ("fp32", 64, 1, 2, 352), ("fp32", 64, 1, 2, 353), ("fp32", 128, 7, 16, 256), ("fp32", 128, 7, 16, 257),
    # sixty splits; seven of four waves; caches as large as the Infinity Cache; a second launch's merge
    ("bf16", 128, 1, 1, 10300), ("bf16", 128, 3, 43, 600), ("fp32", 128, 4, 16, 3841), ("bf16", 64, 3, 100, 1030)])
def test_one_step_from_random_caches(dtype, d, B, H, n, gates):
    import torch
    import paper_2505_16381_amd as pa
    from oracle import decode_oracle
    td = torch.float32 if dtype == "fp32" else torch.bfloat16
    gen = torch.Generator().manual_seed(n + d + H)
    rn = lambda *s: torch.randn(*s, generator=gen)
    q, k, v = (rn(B, H, d).to(td) for _ in range(3))
    w = torch.nn.functional.normalize(rn(B, H, d), dim=-1).to(td)
    beta = (2 * torch.rand(B, H, generator=gen)).to(td)
    log_f = torch.nn.functional.logsigmoid(rn(B, H) + 2).to(td)
    Lmax = n + 3
    kc, vc = rn(B, H, Lmax, d).to(td), rn(B, H, Lmax, d).to(td)
    cc = torch.cumsum(torch.nn.functional.logsigmoid(rn(B, H, Lmax) + 2), -1)
    scale = d ** -0.5
    dev = [t.cuda() for t in (q, k, v, w, beta)]
    gk, gv, gc = kc.cuda(), vc.cuda(), cc.cuda()
    ws = torch.full((pa.path_decode_workspace_bytes(B, H, d),), 255, dtype=torch.uint8, device="cuda")     # NaNs
    if gates:
        o, lse = pa.path_decode_step_fox(*dev, log_f.cuda(), gk, gv, gc, n, scale, workspace=ws)
    else:
        o, lse = pa.path_decode_step(*dev, gk, gv, n, scale, workspace=ws)
    f = lambda t: t.double().cpu().numpy()
    rnd = None if dtype == "fp32" else lambda a: f(torch.from_numpy(a).to(td))
    ref = decode_oracle.decode_step(*(f(t) for t in (q, k, v, w, beta)), f(kc[:, :, :n]), f(vc[:, :, :n]), scale, round_cache=rnd,
                                    **(dict(logf_t=f(log_f), cc=f(cc[:, :, :n])) if gates else {}))
    # fp32: the bars of the other decode tests.  bf16: a refreshed key is rounded once, to half a unit of its 8 significand
    # bits -- 2^-8 of its value -- and near a tie the two sides may round apart by a whole unit, 2^-7; a logit then differs by
    # a fraction of 2^-9 |q| |k| scale for the few such keys; outputs are rounded to bf16
    e_o, e_l = np.abs(f(o) - ref[0]).max(), np.abs(f(lse) - ref[1]).max()
    e_k = (np.abs(f(gk)[:, :, :n + 1] - ref[2]) - (0 if dtype == "fp32" else 2.0 ** -7) * np.abs(ref[2])).max()
    print(f"[decode {dtype} d={d} B={B} H={H} n={n} gates={gates}] max|do|={e_o:.2e} max|dlse|={e_l:.2e} keys {e_k:.2e}", flush=True)
    # outputs shrink with the number of keys (a mean of n values): the bar is a share of the largest one.  bf16: 2^-9 from the
    # rounding of o, and as much again at most from the logits; of 64 splits a single one left out moves o by 5e-2 of it or more
    e_r = e_o / np.abs(ref[0]).max()
    assert e_r <= (1e-4 if dtype == "fp32" else 1e-2) and e_l <= 1e-3 and e_k <= 1e-5
    assert torch.equal(gv[:, :, :n].cpu(), vc[:, :, :n]) and torch.equal(gv[:, :, n].cpu(), v) and torch.equal(gk[:, :, n].cpu(), k)
    assert torch.equal(gk[:, :, n + 1:].cpu(), kc[:, :, n + 1:]) and torch.equal(gv[:, :, n + 1:].cpu(), vc[:, :, n + 1:])
    want_c = cc.clone()
    if gates:
        want_c[:, :, n] = (cc[:, :, n - 1] if n else 0.0) + log_f.float()
    assert torch.equal(gc.cpu(), want_c)
