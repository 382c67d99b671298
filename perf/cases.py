"""Representative workloads of the PaTH attention library, one pass each through its public entry points.

Sizes come from the benchmark configurations (``synth_inputs.CONFIGS``), the benchmark's other workloads and the
tests.  ``listed()`` names the workloads, ``draw()`` gives further ones of the same kinds and ranges; ``prepare()``
makes what a caller holds before the call (seeded inputs on the GPU, the workspace its program keeps), ``run()``
is one pass, ``work()`` the bytes and operations the pass cannot do without.

Kinds of pass
  train    forward + backward of one training step as the training pair (one workspace shared by both)
  blhd     forward + backward as the self-contained calls, on tensors in [B,L,H,d] order (a model's own layout)
  packed   forward + backward of packed sequences of unequal length
  forward  forward only (evaluation)
  prompt   forward of a prompt and the key prefill of the decode caches
  decode   one decoding step: every cached key refreshed in place, attention over the cache, token appended
  ring     one device's share of the sequence-parallel forward: own segment, one hop over an earlier one, result
"""
from __future__ import annotations

import itertools
import math
import random

import torch

import paper_2505_16381_amd as pa

MAX_TOKENS = 1 << 19        # B*H*L of a drawn training step: that of the headline configuration
MAX_PAIRS = 64 * 8192 ** 2  # B*H*L*L of a drawn training step: ditto


def _case(kind, B, H, L, d, dtype="bf16", gates=False, beta_mean=0.0, **more):
    return dict(kind=kind, B=B, H=H, L=L, d=d, dtype=dtype, gates=gates, beta_mean=beta_mean, **more)


def listed():
    return [
        # the headline training step
        dict(name="train_L8192_d128", **_case("train", 4, 16, 8192, 128)),
        # the same with narrow heads and shorter sequences, more of them
        dict(name="train_L4096_d64", **_case("train", 8, 16, 4096, 64)),
        # long-context training: few heads, far keys dominate, beta near 2; the largest pass
        dict(name="train_L32768_d128", **_case("train", 1, 32, 32768, 128, beta_mean=2.0)),
        # a tiny fp32 step (debugging, gradient checks): launches and latency
        dict(name="train_L256_d64_fp32", **_case("train", 1, 2, 256, 64, dtype="fp32")),
        # forget gates, a model's own layout, a ragged length, no workspace kept between forward and backward
        dict(name="blhd_L3000_d128_gates", **_case("blhd", 4, 16, 3000, 128, gates=True)),
        # a packed batch of documents of 256 to 2048 tokens
        dict(name="packed_64_docs_d128", **_case("packed", 64, 8, 2048, 128, shortest=256)),
        # evaluation forward
        dict(name="forward_L2048_d64", **_case("forward", 8, 16, 2048, 64)),
        # a prompt arriving at a server: forward, then the decode caches are filled
        dict(name="prompt_L1000_d128", **_case("prompt", 1, 16, 1000, 128)),
        # decoding over a long cache with a batch: HBM-bound
        dict(name="decode_n8192_d128", **_case("decode", 4, 16, 8192, 128)),
        # decoding with forget gates, narrow heads, a larger batch and an odd cache length
        dict(name="decode_n3001_d64_gates", **_case("decode", 8, 16, 3001, 64, gates=True)),
        # a single sequence early in its decoding: latency
        dict(name="decode_n500_d128", **_case("decode", 1, 16, 500, 128)),
        # one device of a sequence split over several: 4096 tokens each
        dict(name="ring_L4096_d128", **_case("ring", 2, 16, 4096, 128)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: kinds as in listed(), lengths over the whole range on a logarithmic scale (odd ones among
    them), as many heads as the bounds on tokens and on query-key pairs leave room for."""
    kind = rng.choice(["train", "train", "blhd", "packed", "forward", "prompt", "decode", "decode", "ring"])
    d = rng.choice([64, 128])
    gates = rng.random() < 0.3
    if kind == "decode":
        n = _log_int(rng, 64, 32768)
        H = rng.choice([8, 16, 32])
        B = min(_log_int(rng, 1, 32), max(1, (64 * 8192) // (n * H)))
        return _case(kind, B, H, n, d, gates=gates)
    if kind == "packed":
        longest = _log_int(rng, 256, 4096)
        return _case(kind, _log_int(rng, 2, 64), rng.choice([4, 8, 16]), longest, d, gates=gates, shortest=max(1, longest // 8))
    if kind == "prompt":
        L = _log_int(rng, 100, 16384)
        return _case(kind, min(_log_int(rng, 1, 8), max(1, 16384 // L)), rng.choice([8, 16, 32]), L, d)
    if kind == "ring":
        L = 64 * _log_int(rng, 4, 128)      # an earlier segment is a whole number of chunks
        return _case(kind, 1, rng.choice([8, 16, 32]), L, d)
    if kind == "train" and rng.random() < 0.2:      # fp32: small steps only
        return _case(kind, 1, rng.choice([1, 2, 4]), _log_int(rng, 64, 1024), d, dtype="fp32", gates=gates)
    L = _log_int(rng, 128, 16384)
    most = max(1, min(128, MAX_TOKENS // L, MAX_PAIRS // (L * L)))
    heads = _log_int(rng, min(2, most), most)
    H = max(h for h in (1, 2, 4, 8, 16) if h <= heads)
    return _case(kind, max(1, heads // H), H, L, d, gates=gates and kind != "forward")


def _offsets(case):
    """Token offsets of a case's packed sequences: lengths spread uniformly between the shortest and the longest
    (which always occurs), in no order."""
    n, lo, hi = case["B"], case["shortest"], case["L"]
    lens = random.Random(f"{n} {lo} {hi}").choices(range(lo, hi + 1), k=n)
    lens[n // 2] = hi
    return [0, *itertools.accumulate(lens)]


def prepare(case, seed):
    kind, B, H, L, d = case["kind"], case["B"], case["H"], case["L"], case["d"]
    dev = torch.device("cuda")
    td = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    dt = pa.PATH_BF16 if case["dtype"] == "bf16" else pa.PATH_F32
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rn = lambda *shape: torch.randn(*shape, device=dev, generator=gen)
    empty = lambda nbytes: torch.empty(max(256, nbytes), dtype=torch.uint8, device=dev)

    def vectors(*shape):
        """q, k, v, w of one layer: standard normal, w of unit length; beta in (0, 2); log gates of a few per cent."""
        q, k, v = (rn(*shape, d).to(td) for _ in range(3))
        w = torch.nn.functional.normalize(rn(*shape, d), dim=-1).to(td)
        beta = (2 * torch.sigmoid(rn(*shape) + case["beta_mean"])).to(td)
        log_f = torch.nn.functional.logsigmoid(rn(*shape) + 2.0).to(td) if case["gates"] else None
        return dict(q=q, k=k, v=v, w=w, beta=beta, log_f=log_f)

    s = dict(case=case, dt=dt, scale=d ** -0.5)
    if kind == "train":
        s.update(vectors(B, H, L), d_o=rn(B, H, L, d).to(td), ws=empty(pa.path_attn_workspace_bytes(B, H, L, d, dt, True)))
    elif kind == "blhd":
        s.update(vectors(B, L, H), d_o=rn(B, L, H, d).to(td), ws=empty(pa.path_attn_workspace_bytes(B, H, L, d, dt, True)))
    elif kind == "packed":
        cu = _offsets(case)
        T = cu[-1]
        s.update(vectors(T, H), d_o=rn(T, H, d).to(td), cu=cu, ws=empty(pa.path_attn_varlen_workspace_bytes(cu, H, d, dt, True)))
    elif kind in ("forward", "prompt"):
        s.update(vectors(B, H, L), ws=empty(pa.path_attn_workspace_bytes(B, H, L, d, dt, False)))
        if kind == "prompt":      # caches with room for an answer
            s.update(kc=torch.zeros(B, H, L + 256, d, dtype=td, device=dev), vc=torch.zeros(B, H, L + 256, d, dtype=td, device=dev))
    elif kind == "decode":
        s.update(vectors(B, H), kc=rn(B, H, L + 64, d).to(td), vc=rn(B, H, L + 64, d).to(td), ws=empty(pa.path_decode_workspace_bytes(B, H, d)))
        if case["gates"]:
            s["cc"] = torch.cumsum(torch.nn.functional.logsigmoid(rn(B, H, L + 64) + 2.0), -1)
    elif kind == "ring":
        # what a device holds: its own segment, and the tiles of the segment before as received from its neighbour
        s.update(vectors(B, H, L), ws=empty(pa.path_attn_workspace_bytes(B, H, L, d, dt, False)),
                 state=empty(pa.path_attn_ring_state_bytes(B, H, L, d)), remote=empty(pa.path_attn_workspace_bytes(B, H, L, d, dt, False)))
        e = vectors(B, H, L)
        pa.path_attn_ring_local(e["q"], e["k"], e["v"], e["w"], e["beta"], s["state"], s["remote"], scale=s["scale"])
        s["o"], s["lse"] = torch.empty_like(s["q"]), torch.empty(B, H, L, dtype=torch.float32, device=dev)
    else:
        raise ValueError(kind)
    return s


def run(s):
    kind, scale, ws, log_f = s["case"]["kind"], s["scale"], s["ws"], s["log_f"]
    x = (s["q"], s["k"], s["v"], s["w"], s["beta"])
    if kind == "train":
        o, lse = pa.path_attn_train_fwd(*x, ws, log_f=log_f, scale=scale)
        return o, lse, pa.path_attn_train_bwd(*x, o, lse, s["d_o"], ws, log_f=log_f, scale=scale)
    if kind == "blhd":
        o, lse = pa.path_attn_fwd_layout(*x, pa.PATH_LAYOUT_BLHD, log_f=log_f, scale=scale, workspace=ws)
        return o, lse, pa.path_attn_bwd_layout(*x, o, lse, s["d_o"], pa.PATH_LAYOUT_BLHD, log_f=log_f, scale=scale, workspace=ws)
    if kind == "packed":
        o, lse = pa.path_attn_varlen_fwd(*x, s["cu"], log_f=log_f, scale=scale, workspace=ws)
        return o, lse, pa.path_attn_varlen_bwd(*x, o, lse, s["d_o"], s["cu"], log_f=log_f, scale=scale, workspace=ws)
    if kind == "forward":
        return pa.path_attn_fwd(*x, scale=scale, workspace=ws)
    if kind == "prompt":
        o, lse = pa.path_attn_fwd(*x, scale=scale, workspace=ws)
        pa.path_key_prefill(s["v"], ws, s["kc"], s["vc"])
        return o, lse, s["kc"], s["vc"]
    if kind == "decode":
        n = s["case"]["L"]
        if log_f is None:
            o, lse = pa.path_decode_step(*x, s["kc"], s["vc"], n, scale, workspace=ws)
            return o, lse, s["kc"], s["vc"]
        o, lse = pa.path_decode_step_fox(*x, log_f, s["kc"], s["vc"], s["cc"], n, scale, workspace=ws)
        return o, lse, s["kc"], s["vc"], s["cc"]
    # ring
    B, H, L, d = s["q"].shape
    pa.path_attn_ring_local(*x, s["state"], ws, log_f=log_f, scale=scale)
    pa.path_attn_ring_hop(s["state"], B, H, L, s["remote"], L, d, s["dt"], with_gates=log_f is not None, scale=scale)
    pa.path_attn_ring_finish(s["state"], s["o"], s["lse"], gates_workspace=ws if log_f is not None else None)
    return s["o"], s["lse"]


def work(case):
    """Bytes: every input read once, every output written once.  Operations: 4 d per (query, key <= query) pair of
    the forward's logits and P V, 10 d more for the backward's five products (what the method adds is not counted)."""
    kind, B, H, L, d = case["kind"], case["B"], case["H"], case["L"], case["d"]
    es = 2 if case["dtype"] == "bf16" else 4
    g = 1 if case["gates"] else 0
    if kind == "decode":      # keys read and written, values read; per key: w.k, the refresh, q.k, P V
        return {"bytes": B * H * (L * (3 * d * es + 4 * g) + 7 * d * es), "flops": B * H * L * 8.0 * d}
    if kind == "packed":
        cu = _offsets(case)
        tokens, pairs = H * cu[-1], H * sum((b - a) * (b - a + 1) / 2 for a, b in zip(cu, cu[1:]))
    else:
        tokens, pairs = B * H * L, B * H * L * (L + 1) / 2
    fwd_in, fwd_out = tokens * ((4 * d + 1 + g) * es), tokens * (d * es + 4)
    if kind in ("train", "blhd", "packed"):
        bwd_in, bwd_out = tokens * ((6 * d + 1 + g) * es + 4), tokens * ((4 * d + 1 + g) * es)
        return {"bytes": fwd_in + fwd_out + bwd_in + bwd_out, "flops": 14.0 * d * pairs}
    if kind == "prompt":
        return {"bytes": fwd_in + fwd_out + tokens * 2 * d * es, "flops": 4.0 * d * pairs}
    if kind == "ring":        # the earlier segment: keys, values and gate sums; all pairs of the hop
        return {"bytes": fwd_in + fwd_out + tokens * (2 * d * es + 4 * g), "flops": 4.0 * d * (pairs + B * H * L * L)}
    return {"bytes": fwd_in + fwd_out, "flops": 4.0 * d * pairs}


def tolerance(case):
    """Against the fp64 oracle, per output: 1.6e-3 .. 3.3e-3 of the norm with bf16 tensors, at worst 0.08 of the
    output's root mean square; with fp32 tensors up to 6.6e-6 (of which gates and length make the most) and 8e-5.
    Two implementations differ by about as much; about four times that is stated."""
    if case["dtype"] == "fp32":
        return {"rel": 2.5e-5, "max": 5e-4}
    return {"rel": 1e-2, "max": 0.3}
