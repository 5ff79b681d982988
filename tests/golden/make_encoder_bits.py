"""Writes tests/golden/encoder_bits.json: digests of what small encoders give on an MI355X, to the bit -- logits, losses and weights of a batch,
the gradient of a base step, g_meta, v, the hypergradient and the step size of a meta step.  For each length of sequence and
both forms of a batch, on both sides of the sizes at which attention and residuals take other kernels.

The hypergradient is a difference of two nearly equal gradients and magnifies whatever is rounded or added in another order, far
beyond any tolerance of its own, so that a change of a kernel that keeps these bits is the only one that needs no other proof.  The digests are of kernels that round a
probability of attention after its division and add a hi + lo product as 16 of hi, 16 of lo; record them again only with a step that changes rounding on purpose."""
import hashlib
import json
import os
import sys
import numpy as np

ROOT = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "..")
FILE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "encoder_bits.json")
#          B, (L, d, heads, ffn), S, padded
CASES = [(5, (2, 192, 3, 320), 64, False), (7, (2, 192, 3, 320), 64, True), (5, (2, 192, 3, 320), 128, False), (7, (2, 192, 3, 320), 128, True),
         (3, (2, 192, 3, 320), 256, False), (6, (2, 192, 3, 320), 256, True),
         (30, (3, 640, 10, 1280), 128, False), (31, (3, 640, 10, 1280), 128, True)]


def name_of(case):
    B, dims, S, padded = case
    return f"{B} x {S}{' padded' if padded else ''}, {'x'.join(map(str, dims))}"


def encoder_bits(case):
    """{output: digest} of one case."""
    import torch
    import paper_2310_05674_amd as pkg
    from datagen import make_workload, init_theta, init_lambda
    B, dims, S, padded = case
    wl = make_workload(3, n_train=B, n_meta=B, dims=dims + (S, 300, 3), batch=B, meta_batch=B)
    cfg = pkg.SamaConfig.make(wl.kind, wl.dims, H=wl.H, max_batch=B, max_meta_batch=B, base_lr=1e-3, meta_lr=wl.meta_lr, alpha=wl.alpha)
    s = pkg.Sama(cfg, init_theta(wl, 0.02), init_lambda(wl))
    dev = lambda a, t: torch.as_tensor(np.ascontiguousarray(a).astype(t), device=s.dev)
    lens = lambda k: dev(np.clip((np.arange(B) * k) % (2 * S), 1, S), np.int32) if padded else None
    train = s.batch(dev(wl.x_train[:B], np.int32), dev(wl.y_train[:B], np.int32), seq_len=lens(37))
    meta = s.batch(dev(wl.x_meta[:B], np.int32), dev(wl.y_meta[:B], np.int32), seq_len=lens(53))
    got = {k: torch.zeros(n, device=s.dev) for k, n in (("logits", (B, 3)), ("losses", (B,)), ("weights", (B,)))}
    s.eval(train, *got.values())
    for _ in range(2):
        s.base_step(train)
    got["G"] = s.get_state("G")
    s.meta_step(train, meta)
    for k in ("GMETA", "VDIR", "SCALARS", "HYPERGRAD", "THETA"):
        got[k] = s.get_state(k)
    out = {k: hashlib.sha256(v.cpu().numpy().tobytes()).hexdigest()[:16] for k, v in got.items()}
    s.close()
    return out


if __name__ == "__main__":
    sys.path.insert(0, os.path.abspath(ROOT))
    json.dump({name_of(c): encoder_bits(c) for c in CASES}, open(sys.argv[1] if len(sys.argv) > 1 else FILE, "w"), indent=1)
