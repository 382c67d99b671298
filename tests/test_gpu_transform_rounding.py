"""N = A^-1 diag(beta) of the 16-bit chunk transform is rounded once, to the operand type (run with -m gpu).  Three tokens per head, made such that the
last one's log-sum-exp is one element of N, with factors for which a rounding to 32 bits on the way gives the other neighbour of a tie."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
HEADS = 48


def _bf16(rng, lo, hi, n):
    """Random values of eight significant bits."""
    m, e = np.frexp(rng.uniform(lo, hi, n))
    return np.ldexp(np.round(m * 256) / 256, e)


def _factors():
    """w_1 = (a, b, ..), w_2 = (c, e, ..), beta_1, beta_2 of HEADS cases, and the element beta_2 (w_2 . w_1) beta_1 rounded once."""
    rng = np.random.default_rng(11)
    n = 1 << 21
    a, c = _bf16(rng, 0.25, 0.5, n), _bf16(rng, 0.25, 0.5, n)
    b, e = _bf16(rng, 2.0 ** -5, 2.0 ** -4, n), _bf16(rng, 2.0 ** -5, 2.0 ** -4, n)
    b1, b2 = _bf16(rng, 1.0, 1.9, n), _bf16(rng, 1.0, 1.9, n)
    g = a * c + b * e                                       # exact in 32 bits
    assert np.array_equal(g, g.astype(np.float32))
    x = (b2 * g).astype(np.float32).astype(np.float64)      # -(A^-1)_21
    once, twice = (x * b1).astype(np.float16), (x * b1).astype(np.float32).astype(np.float16)
    sel = np.flatnonzero(once != twice)[:HEADS]
    assert sel.size == HEADS
    return [y[sel] for y in (a, b, c, e, b1, b2)], once[sel].astype(np.float64)


@pytest.mark.parametrize("train", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_rounded_once(d, train):
    import torch
    import paper_2505_16381_amd as pa
    (a, b, c, e, b1, b2), want = _factors()
    q, k, v, w = (np.zeros((1, HEADS, 3, d)) for _ in range(4))
    beta = np.zeros((1, HEADS, 3))
    w[0, :, 1, 0], w[0, :, 1, 1], w[0, :, 1, 3] = a, b, 0.5
    w[0, :, 2, 0], w[0, :, 2, 1], w[0, :, 2, 4] = c, e, 0.5
    beta[0, :, 1], beta[0, :, 2] = b1, b2
    k[0, :, 0, 3] = 2                                       # w_1 . k_0 = 1, w_2 . k_0 = 0
    q[0, :, 2, 4] = 2                                       # q_2 . w_2 = 1, q_2 . w_1 = 0, q_2 . k_0 = 0
    q[0, :, 2, 2], k[0, :, 1:, 2] = 30, -30                 # the other two logits: -900
    args = [torch.from_numpy(t).to("cuda").bfloat16().contiguous() for t in (q, k, v, w, beta)]
    if train:
        ws = torch.empty(pa.path_attn_workspace_bytes(1, HEADS, 3, d, pa.PATH_BF16, True), dtype=torch.uint8, device="cuda")
        _, lse = pa.path_attn_train_fwd(*args, ws, scale=1.0)
    else:
        _, lse = pa.path_attn_fwd(*args, scale=1.0)
    got = lse[0, :, 2].double().cpu().numpy()
    assert np.abs(got - want).max() <= 2e-6 * np.abs(want).max()      # (a step of the operand type is 1.9e-4 of it at least)
