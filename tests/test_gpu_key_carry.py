"""Key prefill on both sides of the rule that carries every chunk by itself (16-bit operands; run with -m gpu): few heads and
many, one block to pass, several, none, ragged last chunks, against the decode oracle on the first and the last head."""
import numpy as np
import pytest

from paper_2505_16381_amd import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,L,H", [(128, 64, 9), (64, 130, 3), (128, 1024, 2), (128, 700, 100), (64, 1000, 200), (128, 1025, 3), (128, 1025, 150),
                                   (64, 3200, 5), (64, 3200, 120), (128, 2300, 7)])
def test_keys_at_the_prompts_end(d, L, H):
    import torch
    import paper_2505_16381_amd as pa
    from oracle import decode_oracle
    x = si.make_inputs(1, 2, L, d, "bf16", 31 + L + d, 0.0)
    # heads 0 and H - 1 are the oracle's, the ones between repeat them
    idx = [0] + [i % 2 for i in range(1, H - 1)] + [1]
    dv = {n: torch.from_numpy(np.ascontiguousarray(a[:, idx])).to("cuda").to(torch.bfloat16) for n, a in x.items()}
    ws = torch.full((pa.path_attn_workspace_bytes(1, H, L, d, pa.PATH_BF16, False),), 255, dtype=torch.uint8, device="cuda")      # NaNs
    pa.path_attn_fwd_prep(dv["q"], dv["k"], dv["v"], dv["w"], dv["beta"], ws)
    kc = torch.full((1, H, L + 5, d), 7.0, dtype=torch.bfloat16, device="cuda")
    vc = kc.clone()
    pa.path_key_prefill(dv["v"], ws, kc, vc)
    want = decode_oracle.key_prefill(x["k"], x["w"], x["beta"])
    got = kc[:, [0, H - 1], :L].float().cpu().numpy()
    # bf16 rounds a key to 2^-9 of it; half as much again for the transport (the bar of the other prefill tests)
    assert np.abs(got - want).max() <= 2.0 ** -8 * np.abs(want).max() * 1.5
    for h in range(1, H - 1):
        assert torch.equal(kc[:, h], kc[:, 0 if idx[h] == 0 else H - 1])
    assert torch.equal(vc[:, :, :L], dv["v"]) and bool((kc[:, :, L:] == 7).all()) and bool((vc[:, :, L:] == 7).all())
