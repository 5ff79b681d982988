"""GPU parity, bf16 encoder workloads: the HIP path through the C ABI against the float64 oracle on the same
seeded inputs, from the oracle's unrounded state (teacher-forced) and free-running.  Bar: relative L2 <= 2e-2 on the
hypergradient and the updated theta / lambda (bf16 GEMM operands, fp32 accumulation and state).  Nothing in this file
rounds the oracle's state to what the kernels can hold, except the one test of the mixed-precision switch
(fast_base_pass = 1), which says so."""
import numpy as np
import pytest
from datagen import make_workload, init_theta, init_lambda, round_to_bf16, seq_lengths
from oracle.models import with_lengths
from harness import rel_l2, make_pair, dev_batch, push_state, pull

pytestmark = pytest.mark.gpu
TOL = 2e-2

SMALL = dict(dims=(2, 192, 3, 320, 128, 600, 3), batch=5, meta_batch=3)      # ragged N tiles, odd batch sizes
KTOL = 1e-2     # bar of the small-shape tests on single gradients: ~10 bf16 roundings (2^-9) of GEMM inputs per layer


def _well_measured(orc, tau=0.1):
    """Entries whose kept base gradient lies above the noise floor of a bf16 pass: |g_i| >= tau * rms of g over the
    entry's tensor (from the oracle alone).  A pass with bf16 GEMM operands carries an error of the order of 1e-3 of a
    tensor's rms on EVERY entry of its gradient, so the relative error of an entry grows as the entry shrinks -- and the
    adaptation of Eq. 4 is largest (by orders of magnitude) exactly on the entries with the smallest gradient history,
    which therefore hold most of ||v||^2 while being the worst measured.  With the GPU's own g, m', v' in Eq. 4 the
    perturbation vector is compared entry by entry on the well-measured entries; its norm enters through eps."""
    mask = np.zeros(orc.g.size, dtype=bool)
    for name, (off, shape) in orc.model.slices.items():
        sl = slice(off, off + int(np.prod(shape)))
        mask[sl] = np.abs(orc.g[sl]) >= tau * np.sqrt(np.mean(orc.g[sl] ** 2))
    return mask


def _gemm_block(orc):
    return sum(int(np.prod(sh)) for nm, (o, sh) in orc.model.slices.items() if nm.split(".")[-1] in ("Wqkv", "Wo", "W1", "W2"))


def _batches(wl, step):
    it, im = wl.train_batch(step), wl.meta_batch_idx(step)
    return (wl.x_train[it], wl.y_train[it]), (wl.x_meta[im], wl.y_meta[im])


def _group_errors(orc, got, want):
    out = {}
    for name, (off, shape) in orc.model.slices.items():
        sl = slice(off, off + int(np.prod(shape)))
        out[name] = rel_l2(got[sl], want[sl])
    return out


@pytest.mark.parametrize("scale", [0.02, 0.08])
def test_small_encoder_base_step(scale):
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    orc, gpu = make_pair(wl, init_theta(wl, scale), init_lambda(wl), base_lr=1e-3)
    for s in range(2):
        (x, y), _ = _batches(wl, s)
        push_state(orc, gpu)
        th_before = orc.theta.copy()
        l_before = orc.model.losses(orc.theta, x, y)
        lo = orc.base_step(x, y)
        gpu.base_step(dev_batch(gpu, x, y))
        losses = pull(gpu, "LOSSES")[:len(y)]
        # diagnostic: how much of the difference is the bf16 rounding of the GEMM weights themselves
        ng = sum(int(np.prod(sh)) for nm, (o, sh) in orc.model.slices.items() if nm.split(".")[-1] in ("Wqkv", "Wo", "W1", "W2"))
        th_r = th_before.copy(); th_r[:ng] = round_to_bf16(th_r[:ng])
        l_r = orc.model.losses(th_r, x, y)
        print(f"  losses: max|l|={np.max(l_before):.3f} gpu-oracle {np.max(np.abs(losses - l_before)):.2e} "
              f"gpu-oracle(bf16 weights) {np.max(np.abs(losses - l_r)):.2e}")
        assert np.max(np.abs(losses - l_before)) < 2e-2 * max(1.0, np.max(l_before)), np.max(np.abs(losses - l_before))
        g = pull(gpu, "G")
        errs = _group_errors(orc, g, orc.g)
        worst = max(errs, key=errs.get)
        print(f"scale {scale} step {s}: rel-L2 g {rel_l2(g, orc.g):.3e}; worst group {worst} {errs[worst]:.3e}")
        assert rel_l2(g, orc.g) < KTOL
        assert all(e < 2e-2 for e in errs.values()), errs
        assert rel_l2(pull(gpu, "THETA"), orc.theta) < TOL
        assert abs(float(pull(gpu, "SCALARS")[2]) - lo) < 2e-2 * abs(lo)
    gpu.close()


@pytest.mark.parametrize("scale", [0.02, 0.08])
def test_small_encoder_meta_step(scale):
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    orc, gpu = make_pair(wl, init_theta(wl, scale), init_lambda(wl), base_lr=1e-3)
    for s in range(3):
        (x, y), _ = _batches(wl, s)
        orc.base_step(x, y)
    for s in range(3, 5):
        (x, y), (xm, ym) = _batches(wl, s)
        orc.base_step(x, y)
        push_state(orc, gpu)
        tb, mb = dev_batch(gpu, x, y), dev_batch(gpu, xm, ym)
        r = orc.meta_step(x, y, xm, ym)
        gpu.meta_step(tb, mb)
        h = pull(gpu, "HYPERGRAD")
        e = dict(gmeta=rel_l2(pull(gpu, "GMETA"), r["g_meta"]), v=rel_l2(pull(gpu, "VDIR"), r["v"]),
                 eps=abs(pull(gpu, "SCALARS")[0] - r["eps"]) / r["eps"], h=rel_l2(h, r["h"]),
                 glam_p=rel_l2(pull(gpu, "GLAM_PLUS"), r["glam_p"]), theta=rel_l2(pull(gpu, "THETA"), orc.theta),
                 lam=rel_l2(pull(gpu, "LAMBDA"), orc.lam))
        print(f"scale {scale} step {s}: " + " ".join(f"{k}={v:.2e}" for k, v in e.items()))
        assert e["gmeta"] < KTOL and e["glam_p"] < KTOL and e["eps"] < KTOL and e["v"] < TOL
        # at scale 0.08 / lr 1e-3 the map v -> h is ill-conditioned (a 1e-2 change of v moves h by 4e-2 in exact
        # arithmetic as well), so there h is printed, not asserted: its inputs (g_meta, v, eps, g_lambda^+) carry the bars
        if scale == 0.02:
            assert e["h"] < TOL, e
        assert e["theta"] < TOL and e["lam"] < TOL
        assert int(pull(gpu, "COUNTERS")[2]) == 0
    gpu.close()


def test_meta_grad_is_pure_and_matches_meta_step():
    """sama_meta_grad leaves theta, lambda and the moments untouched and returns the hypergradient that sama_meta_step
    then applies.  The two take different routes through the elementwise chain (separate low halves and nudge against
    the old bf16 copy / one fused pass against the new one), so the two hypergradients agree to rounding of the low
    halves, not bit for bit; the applied step must still land on the oracle's theta."""
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    for s in range(4):
        (x, y), _ = _batches(wl, s)
        orc.base_step(x, y)
    (x, y), (xm, ym) = _batches(wl, 4)
    push_state(orc, gpu)
    tb, mb = dev_batch(gpu, x, y), dev_batch(gpu, xm, ym)
    before = {k: pull(gpu, k).copy() for k in ("THETA", "LAMBDA", "M", "V", "META_M", "META_V")}
    gpu.meta_grad(tb, mb)
    for k, v in before.items():
        assert np.array_equal(pull(gpu, k), v), k
    h_pure = pull(gpu, "HYPERGRAD").copy()
    gpu.meta_grad(tb, mb)
    assert np.array_equal(pull(gpu, "HYPERGRAD"), h_pure)          # and is repeatable bit for bit
    r = orc.meta_step(x, y, xm, ym)
    gpu.meta_step(tb, mb)
    h = pull(gpu, "HYPERGRAD")
    assert rel_l2(h_pure, r["h"]) < TOL and rel_l2(h, r["h"]) < TOL
    assert rel_l2(h, h_pure) < 5e-3, rel_l2(h, h_pure)
    assert rel_l2(pull(gpu, "THETA"), orc.theta) < TOL
    th = pull(gpu, "THETA")
    # the nudge itself, fused block and tail alike: theta_old - eps v with the GPU's own eps and v, one fp32 rounding
    want = before["THETA"].astype(np.float64) - float(pull(gpu, "SCALARS")[0]) * pull(gpu, "VDIR").astype(np.float64)
    assert np.max(np.abs(th - want)) <= 2.0 ** -23 * np.max(np.abs(want))
    for name, (off, shape) in orc.model.slices.items():           # every tensor moved, GEMM block and tail alike
        sl = slice(off, off + int(np.prod(shape)))
        assert not np.array_equal(th[sl], before["THETA"][sl]), name
    gpu.close()


# ------------------------------------------------------------------------------------------ full workloads 3-5
_RUNS = {}


def _run_workload(cfg, n_train, n_meta):
    """Real shapes and hyper-parameters of workload `cfg`, nothing rounded anywhere; one run per workload serves the
    tests below (the oracle takes a minute on workload 5).
      a. base step 0 from the initial theta on both sides: the gradient of one pass;
      b. one more oracle base step (history for the adaptation), its state pushed, one meta step (teacher-forced);
      c. the oracle's state after that meta step -- a general point: fp32 master weights off the bf16 grid after two
         Adam steps and a nudge -- pushed once, then ONE WHOLE ITERATION on each side from its own state: base step
         (gradient compared), then the meta step with the GPU's own g, m', v' in the adaptation of Eq. 4."""
    if cfg in _RUNS:
        return _RUNS[cfg]
    import time
    t0 = time.time()
    wl = make_workload(cfg, n_train=n_train, n_meta=n_meta)
    orc, gpu = make_pair(wl, init_theta(wl), init_lambda(wl))
    out = {}
    (x, y), _ = _batches(wl, 0)
    orc.base_step(x, y)
    gpu.base_step(dev_batch(gpu, x, y))
    g = pull(gpu, "G")
    errs = _group_errors(orc, g, orc.g)
    worst = max(errs, key=errs.get)
    out["a"] = dict(g=rel_l2(g, orc.g), worst=errs[worst], theta=rel_l2(pull(gpu, "THETA"), orc.theta))
    print(f"cfg {cfg} a: base step 0 rel-L2 g {out['a']['g']:.3e}, worst group {worst} {errs[worst]:.1e}  [{time.time() - t0:.0f}s]", flush=True)

    def meta_errors(r):
        e = dict(gmeta=rel_l2(pull(gpu, "GMETA"), r["g_meta"]), v=rel_l2(pull(gpu, "VDIR"), r["v"]),
                 eps=abs(pull(gpu, "SCALARS")[0] - r["eps"]) / r["eps"], h=rel_l2(pull(gpu, "HYPERGRAD"), r["h"]),
                 theta=rel_l2(pull(gpu, "THETA"), orc.theta), lam=rel_l2(pull(gpu, "LAMBDA"), orc.lam))
        e["fd_signal"] = np.linalg.norm(r["glam_p"] - r["glam_m"]) / np.linalg.norm(r["glam_p"])
        e["glam_p"] = rel_l2(pull(gpu, "GLAM_PLUS"), r["glam_p"])
        e["status"] = int(pull(gpu, "COUNTERS")[2])
        return e

    (x, y), (xm, ym) = _batches(wl, 1)
    orc.base_step(x, y)
    push_state(orc, gpu)
    r = orc.meta_step(x, y, xm, ym)
    gpu.meta_step(dev_batch(gpu, x, y), dev_batch(gpu, xm, ym))
    out["b"] = meta_errors(r)
    print(f"cfg {cfg} b: " + " ".join(f"{k}={v:.2e}" for k, v in out["b"].items()) + f"  [{time.time() - t0:.0f}s]", flush=True)

    push_state(orc, gpu)
    ng = _gemm_block(orc)
    out["off_grid"] = float(np.mean(round_to_bf16(orc.theta[:ng]) != orc.theta[:ng]))
    (x, y), (xm, ym) = _batches(wl, 2)
    tb, mb = dev_batch(gpu, x, y), dev_batch(gpu, xm, ym)
    th_before = orc.theta.copy()
    orc.base_step(x, y)
    gpu.base_step(tb)
    g = pull(gpu, "G")
    errs = _group_errors(orc, g, orc.g)
    worst = max(errs, key=errs.get)
    out["c_base"] = dict(g=rel_l2(g, orc.g), worst=errs[worst], theta=rel_l2(pull(gpu, "THETA"), orc.theta),
                         step=rel_l2(pull(gpu, "THETA").astype(np.float64) - th_before, orc.theta - th_before),
                         m=rel_l2(pull(gpu, "M"), orc.m), v=rel_l2(pull(gpu, "V"), orc.v))
    print(f"cfg {cfg} c: off-grid weights {out['off_grid']:.2f}; base step rel-L2 g {out['c_base']['g']:.3e} worst group {worst} "
          f"{errs[worst]:.1e} update {out['c_base']['step']:.2e}  [{time.time() - t0:.0f}s]", flush=True)
    well = _well_measured(orc)             # from the oracle's kept gradient, before the meta step moves anything
    r = orc.meta_step(x, y, xm, ym)
    gpu.meta_step(tb, mb)
    out["c_meta"] = meta_errors(r)
    out["c_meta"]["v_well"] = rel_l2(pull(gpu, "VDIR")[well], r["v"][well])
    out["c_meta"]["well_frac"] = float(well.mean())
    out["c_meta"]["well_share"] = float(np.sum(r["v"][well] ** 2) / np.sum(r["v"] ** 2))
    print(f"cfg {cfg} c: " + " ".join(f"{k}={v:.2e}" for k, v in out["c_meta"].items()) + f"  [{time.time() - t0:.0f}s]", flush=True)
    gpu.close()
    _RUNS[cfg] = out
    return out


SIZES = {3: (128, 64), 4: (96, 64), 5: (48, 32)}


@pytest.mark.parametrize("cfg", [3, 4, 5])
def test_workload_parity(cfg):
    """Steps a and b of _run_workload: the gradient of the first base step, and a teacher-forced meta step."""
    o = _run_workload(cfg, *SIZES[cfg])
    assert o["a"]["g"] < KTOL and o["a"]["worst"] < 3e-2 and o["a"]["theta"] < TOL, o["a"]
    e = o["b"]
    assert e["h"] < TOL and e["theta"] < TOL and e["lam"] < TOL and e["eps"] < TOL and e["gmeta"] < TOL and e["v"] < TOL, e
    assert e["status"] == 0


@pytest.mark.parametrize("cfg", [3, 4, 5])
def test_workload_iteration_from_general_state(cfg):
    """Step c of _run_workload: one whole iteration (sama_base_step, then sama_meta_step with the GPU's own gradient and
    moments) from master weights that are NOT bf16-representable, against the oracle doing the same two calls."""
    o = _run_workload(cfg, *SIZES[cfg])
    assert o["off_grid"] > 0.5, o["off_grid"]            # the state really is a general one
    b = o["c_base"]
    assert b["g"] < TOL and b["worst"] < 5e-2 and b["theta"] < TOL and b["step"] < TOL and b["m"] < TOL and b["v"] < TOL, b
    e = o["c_meta"]
    assert e["h"] < TOL and e["theta"] < TOL and e["lam"] < TOL and e["eps"] < TOL and e["gmeta"] < TOL, e
    # v with the GPU's own g, m', v' in Eq. 4: asserted on the entries whose gradient is above the pass's noise floor (see
    # _well_measured: 40-60 % of the entries, which hold only a few per cent of ||v||^2); over all entries it is printed
    # (1e-2 ... 1e-1 depending on the data seed) and enters the assertions through eps, h and theta
    assert e["well_frac"] > 0.3 and e["v_well"] < TOL, e
    assert e["status"] == 0


def test_mixed_precision_switch_sees_the_rounded_weights():
    """fast_base_pass = 1 is ordinary mixed precision: the base step differentiates at bf16(theta).  From a
    bf16-representable theta it agrees with the default (split) pass and with the oracle; from a general state its
    gradient equals the oracle's gradient AT THE ROUNDED WEIGHTS (the only place in this file where oracle weights are
    rounded, to state what the switch computes), while the default pass follows the oracle at theta itself."""
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    th0 = init_theta(wl, 0.02)
    orc, fast = make_pair(wl, th0, init_lambda(wl), base_lr=1e-3, fast_base_pass=1)
    _, split = make_pair(wl, th0, init_lambda(wl), base_lr=1e-3)
    for s in range(3):
        (x, y), _ = _batches(wl, s)
        orc.base_step(x, y)
    (x, y), _ = _batches(wl, 3)
    push_state(orc, fast); push_state(orc, split)
    ng = _gemm_block(orc)
    th_r = orc.theta.copy(); th_r[:ng] = round_to_bf16(th_r[:ng])
    target = orc.targets(th_r, x, y)
    l = orc.model.losses(th_r, x, target)
    from oracle import wnet
    coef = wnet.weights(l, orc.lam) / len(y)
    _, g_rounded = orc.model.loss_grad(th_r, x, target, coef)
    orc.base_step(x, y)
    tb = dev_batch(fast, x, y)
    fast.base_step(tb); split.base_step(dev_batch(split, x, y))
    e_fast_r, e_fast, e_split = rel_l2(pull(fast, "G"), g_rounded), rel_l2(pull(fast, "G"), orc.g), rel_l2(pull(split, "G"), orc.g)
    print(f"fast vs oracle at bf16(theta) {e_fast_r:.2e}; fast vs oracle at theta {e_fast:.2e}; split vs oracle at theta {e_split:.2e}")
    assert e_fast_r < KTOL and e_split < KTOL
    fast.close(); split.close()


# ------------------------------------------------------------------------------------------ unroll > 1
@pytest.mark.parametrize("where", ["small", "workload3"])
def test_unrolled_iteration_free_running(where):
    """Unroll U = 3 (the paper runs U = 10, App. B): three free-running base steps and one meta step on each side from the
    same start, no state pushed in between; a second iteration follows on the small encoder.

    Asserted at the bars of this file: every base step's gradient, moments and weights, the direct gradient, and the
    quantities the parity target names -- hypergradient, theta, lambda.  The perturbation vector v and the step size
    eps are printed only: free-running from zero moments they are ill-conditioned in the method itself.  The adaptation
    of Eq. 4 (App. C) vanishes identically at t = 1, cancels to a tenth of its terms at t = 2, 3, and peaks at
    lr c1 (1 - beta1) / (4 eps_A) for entries with c2 sqrt(v') near eps_A = 1e-8 (pinned in closed form in
    tests/test_oracle_optim.py), i.e. on the few entries whose gradient history is far below the rounding noise of any
    finite-precision pass; in the float64 oracle itself a relative gradient noise of 1e-3 moves v by more than its norm
    there.  The small encoder therefore runs with eps_A = 1e-5, where that peak is a thousand times lower."""
    if where == "small":
        wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
        orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3, adam_eps=1e-5)
        iters = 2
    else:
        wl = make_workload(3, n_train=128, n_meta=64)
        orc, gpu = make_pair(wl, init_theta(wl), init_lambda(wl))
        iters = 1
    k = 0
    for it in range(iters):
        for u in range(3):
            (x, y), (xm, ym) = _batches(wl, k); k += 1
            tb = dev_batch(gpu, x, y)
            orc.base_step(x, y); gpu.base_step(tb)
            e = dict(g=rel_l2(pull(gpu, "G"), orc.g), theta=rel_l2(pull(gpu, "THETA"), orc.theta),
                     m=rel_l2(pull(gpu, "M"), orc.m), v=rel_l2(pull(gpu, "V"), orc.v))
            print(f"{where} it {it} base step {u}: " + " ".join(f"{kk}={vv:.2e}" for kk, vv in e.items()))
            assert e["g"] < KTOL and e["theta"] < TOL and e["m"] < KTOL and e["v"] < KTOL, e
        r = orc.meta_step(x, y, xm, ym)
        gpu.meta_step(tb, dev_batch(gpu, xm, ym))
        e = dict(gmeta=rel_l2(pull(gpu, "GMETA"), r["g_meta"]), v=rel_l2(pull(gpu, "VDIR"), r["v"]),
                 eps=abs(pull(gpu, "SCALARS")[0] - r["eps"]) / r["eps"], h=rel_l2(pull(gpu, "HYPERGRAD"), r["h"]),
                 theta=rel_l2(pull(gpu, "THETA"), orc.theta), lam=rel_l2(pull(gpu, "LAMBDA"), orc.lam))
        print(f"{where} it {it} meta step: " + " ".join(f"{kk}={vv:.2e}" for kk, vv in e.items()))
        assert e["gmeta"] < KTOL and e["h"] < TOL and e["theta"] < TOL and e["lam"] < TOL, e
        if where == "small":       # well-conditioned there (eps_A = 1e-5): the direction and the step size carry bars too
            assert e["v"] < TOL and e["eps"] < KTOL, e
        assert int(pull(gpu, "COUNTERS")[0]) == 3 * (it + 1) and int(pull(gpu, "COUNTERS")[1]) == it + 1
        assert int(pull(gpu, "COUNTERS")[2]) == 0
    gpu.close()


def test_second_stream_changes_no_result():
    """The backward pass runs its weight-gradient launches, and the per-layer optimizer update / adaptation behind them,
    on a second stream.  With everything on one stream instead (tuning hooks of the library) a base step must give the
    same bits, and a meta step the same numbers up to the order in which the partial sums of ||v||^2 are added."""
    import ctypes
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    res = {}
    for mode in (0, 1):
        orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
        gpu.lib.sama_dev_side_stream(ctypes.c_int32(2 * mode)); gpu.lib.sama_dev_side_sink(ctypes.c_int32(mode))   # 2: also for a pass this small
        try:
            for s in range(3):
                (x, y), (xm, ym) = _batches(wl, s)
                gpu.base_step(dev_batch(gpu, x, y))
            after_base = {k: pull(gpu, k).copy() for k in ("G", "THETA", "M", "V")}
            gpu.meta_step(dev_batch(gpu, x, y), dev_batch(gpu, xm, ym))
            res[mode] = (after_base, {k: pull(gpu, k).copy() for k in ("GMETA", "VDIR", "HYPERGRAD", "THETA", "LAMBDA", "SCALARS")})
        finally:
            gpu.lib.sama_dev_side_stream(ctypes.c_int32(1)); gpu.lib.sama_dev_side_sink(ctypes.c_int32(1))
            gpu.close()
    for k in res[0][0]:
        assert np.array_equal(res[0][0][k], res[1][0][k]), k
    assert np.array_equal(res[0][1]["GMETA"], res[1][1]["GMETA"])
    assert np.array_equal(res[0][1]["VDIR"], res[1][1]["VDIR"])
    assert abs(res[0][1]["SCALARS"][0] - res[1][1]["SCALARS"][0]) <= 1e-6 * res[0][1]["SCALARS"][0]
    for k in ("HYPERGRAD", "THETA", "LAMBDA"):
        assert rel_l2(res[1][1][k], res[0][1][k]) < 1e-4, k


def _update_launches(gpu, batch):
    """Launches of the Adam kernel in one base step: one on one stream; on two streams a layer's two ranges follow its
    gradients and the rest comes behind them."""
    gpu.profile(True)
    try:
        gpu.base_step(batch)
        return gpu.profile_read()["adam"][0]
    finally:
        gpu.profile(False)


def test_second_stream_switch_returns_to_the_default():
    """sama_dev_side_stream: 0 keeps one stream, 2 takes two for any size, and 1 is the default again, which for a pass of
    640 rows through two small layers is one stream; so is every value that is not one of the three."""
    import ctypes
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    _, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    (x, y), _ = _batches(wl, 0)
    tb = dev_batch(gpu, x, y)
    try:
        seen = [(-2, _update_launches(gpu, tb))]       # untouched
        for mode in (0, 1, 2, 1, 2, -1):
            gpu.lib.sama_dev_side_stream(ctypes.c_int32(mode))
            seen.append((mode, _update_launches(gpu, tb)))
    finally:
        gpu.lib.sama_dev_side_stream(ctypes.c_int32(1))
        gpu.close()
    print(seen)
    assert all((n > 2 * wl.dims[0]) if mode == 2 else (n == 1) for mode, n in seen), seen


@pytest.mark.parametrize("L,d,B,two", [
    (1, 512, 32, False), (12, 384, 4, False), (2, 192, 8, False), (2, 192, 48, True), (4, 256, 32, True)])
def test_second_stream_by_default(L, d, B, two):
    """Which models take the second stream when nobody asks: a single layer never does, of several those whose rows and layers
    are worth it (both sides of the line, sizes that were measured), and a base step's bits are those of either form."""
    import ctypes
    import paper_2310_05674_amd as pkg
    wl = make_workload(3, n_train=2 * B, n_meta=4, dims=(L, d, d // 64, 4 * d, 128, 600, 3), batch=B, meta_batch=2)
    cfg = pkg.SamaConfig.make(wl.kind, wl.dims, H=wl.H, max_batch=B, max_meta_batch=2, base_lr=1e-3)
    th, lam = init_theta(wl, 0.02), init_lambda(wl)
    (x, y), _ = _batches(wl, 0)
    out, launches = {}, {}
    try:
        for mode in (1, 0, 2):
            gpu = pkg.Sama(cfg, th, lam)
            gpu.lib.sama_dev_side_stream(ctypes.c_int32(mode))
            launches[mode] = _update_launches(gpu, dev_batch(gpu, x, y))
            out[mode] = {k: pull(gpu, k).copy() for k in ("G", "THETA", "M", "V")}
            gpu.close()
    finally:
        gpu.lib.sama_dev_side_stream(ctypes.c_int32(1))
    assert launches[0] < launches[2] and launches[1] == launches[2 if two else 0], launches
    for k in out[1]:
        assert np.array_equal(out[0][k], out[1][k]) and np.array_equal(out[0][k], out[2][k]), k


def test_single_sequence_batches():
    """One train sequence and one meta sequence (M = 128 token rows: a single partial GEMM tile row)."""
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    (x, y), (xm, ym) = _batches(wl, 0)
    x, y, xm, ym = x[:1], y[:1], xm[:1], ym[:1]
    for _ in range(2):
        orc.base_step(x, y)
    push_state(orc, gpu)
    orc.base_step(x, y); gpu.base_step(dev_batch(gpu, x, y))
    assert rel_l2(pull(gpu, "G"), orc.g) < KTOL
    push_state(orc, gpu)
    r = orc.meta_step(x, y, xm, ym)
    gpu.meta_step(dev_batch(gpu, x, y), dev_batch(gpu, xm, ym))
    e = dict(gmeta=rel_l2(pull(gpu, "GMETA"), r["g_meta"]), v=rel_l2(pull(gpu, "VDIR"), r["v"]),
             glam_p=rel_l2(pull(gpu, "GLAM_PLUS"), r["glam_p"]), h=rel_l2(pull(gpu, "HYPERGRAD"), r["h"]),
             theta=rel_l2(pull(gpu, "THETA"), orc.theta), lam=rel_l2(pull(gpu, "LAMBDA"), orc.lam))
    print("single sequence: " + " ".join(f"{k}={v:.2e}" for k, v in e.items()))
    assert e["gmeta"] < KTOL and e["glam_p"] < KTOL and e["v"] < TOL and e["theta"] < TOL and e["lam"] < TOL
    assert e["h"] < TOL, e
    gpu.close()


@pytest.mark.usefixtures("backward_streams")
def test_free_running_trajectory_is_reproducible_bit_for_bit():
    """No floating-point atomics and a fixed order in every reduction, on one stream and on two: two runs of the same 30
    iterations (unroll 2) from the same start end in the same bits."""
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    outs = []
    for rep in range(2):
        _, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
        for k in range(30):
            (x, y), (xm, ym) = _batches(wl, k)
            tb, mb = dev_batch(gpu, x, y), dev_batch(gpu, xm, ym)
            gpu.base_step(tb); gpu.base_step(tb); gpu.meta_step(tb, mb)
        outs.append({k: pull(gpu, k).copy() for k in ("THETA", "LAMBDA", "M", "V", "HYPERGRAD", "COUNTERS")})
        gpu.close()
    assert int(outs[0]["COUNTERS"][0]) == 60 and int(outs[0]["COUNTERS"][1]) == 30 and int(outs[0]["COUNTERS"][2]) == 0
    assert np.all(np.isfinite(outs[0]["THETA"]))
    for k in outs[0]:
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.usefixtures("backward_streams")
@pytest.mark.parametrize("variant", ["sgd", "sgd_momentum", "sama_na"])
def test_small_encoder_sgd_and_no_adaptation(variant):
    """The bf16 encoder with an SGD base solver (D = base lr) and with the adaptation switched off (SAMA-NA, D = 1):
    the per-layer update / adaptation slices of the two-stream backward take their other branches here."""
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    kw = {"sgd": dict(base_opt="sgd", base_lr=0.05), "sgd_momentum": dict(base_opt="sgd", base_lr=0.02, momentum=0.9),
          "sama_na": dict(adapt_mode=1, base_lr=1e-3)}[variant]
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), **kw)
    for s in range(2):
        (x, y), _ = _batches(wl, s)
        orc.base_step(x, y)
    (x, y), (xm, ym) = _batches(wl, 2)
    push_state(orc, gpu)
    th_before = orc.theta.copy()
    orc.base_step(x, y); gpu.base_step(dev_batch(gpu, x, y))
    assert rel_l2(pull(gpu, "G"), orc.g) < KTOL
    assert rel_l2(pull(gpu, "THETA"), orc.theta) < TOL
    if variant != "sama_na":       # SGD's update is linear in g (Adam's divides by sqrt(v'), which magnifies the error of small entries)
        assert rel_l2(pull(gpu, "THETA").astype(np.float64) - th_before, orc.theta - th_before) < KTOL
    if variant == "sgd_momentum":
        assert rel_l2(pull(gpu, "M"), orc.m) < KTOL and rel_l2(orc.m, orc.g) > 0.5                       # the velocity, with history
    push_state(orc, gpu)
    r = orc.meta_step(x, y, xm, ym)
    gpu.meta_step(dev_batch(gpu, x, y), dev_batch(gpu, xm, ym))
    e = dict(gmeta=rel_l2(pull(gpu, "GMETA"), r["g_meta"]), v=rel_l2(pull(gpu, "VDIR"), r["v"]),
             eps=abs(pull(gpu, "SCALARS")[0] - r["eps"]) / r["eps"], h=rel_l2(pull(gpu, "HYPERGRAD"), r["h"]),
             theta=rel_l2(pull(gpu, "THETA"), orc.theta), lam=rel_l2(pull(gpu, "LAMBDA"), orc.lam))
    print(f"{variant}: " + " ".join(f"{k}={v:.2e}" for k, v in e.items()))
    assert e["gmeta"] < KTOL and e["v"] < KTOL and e["eps"] < KTOL and e["h"] < TOL and e["theta"] < TOL and e["lam"] < TOL
    gpu.close()


@pytest.mark.usefixtures("backward_streams")
def test_padded_batches_small_encoder():
    """Sequence lengths (key-padding mask): base step and meta step against the oracle on a length mix that includes a
    one-token and a full sequence; then the invariants of padding on the GPU alone: full lengths give the bits of no
    lengths, and other tokens in the padded positions change no bit of the gradient."""
    import torch
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    S, V = wl.dims[4], wl.dims[5]
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    lens_all = seq_lengths(wl.seed + 1, 64, S)
    for s in range(3):
        (x, y), _ = _batches(wl, s)
        orc.base_step(with_lengths(x, lens_all[5 * s:5 * s + 5]), y)
    for s in range(3, 5):
        (x, y), (xm, ym) = _batches(wl, s)
        lt = lens_all[5 * s:5 * s + 5].copy(); lm = lens_all[40 + 3 * s:43 + 3 * s].copy()
        lt[0], lt[1], lm[0] = 1, S, 2
        push_state(orc, gpu)
        tb, mb = dev_batch(gpu, x, y, lens=lt), dev_batch(gpu, xm, ym, lens=lm)
        # the mask matters on these batches
        assert np.max(np.abs(orc.model.losses(orc.theta, x, y) - orc.model.losses(orc.theta, with_lengths(x, lt), y))) > 1e-3
        lo = orc.base_step(with_lengths(x, lt), y)
        gpu.base_step(tb)
        g = pull(gpu, "G")
        errs = _group_errors(orc, g, orc.g)
        print(f"padded base step {s}: rel-L2 g {rel_l2(g, orc.g):.3e}; worst group {max(errs, key=errs.get)} {max(errs.values()):.3e}")
        assert rel_l2(g, orc.g) < KTOL and all(e < TOL for e in errs.values()), errs
        assert abs(float(pull(gpu, "SCALARS")[2]) - lo) < 2e-2 * abs(lo)
        push_state(orc, gpu)
        r = orc.meta_step(with_lengths(x, lt), y, with_lengths(xm, lm), ym)
        gpu.meta_step(tb, mb)
        e = dict(gmeta=rel_l2(pull(gpu, "GMETA"), r["g_meta"]), h=rel_l2(pull(gpu, "HYPERGRAD"), r["h"]),
                 glam_p=rel_l2(pull(gpu, "GLAM_PLUS"), r["glam_p"]), theta=rel_l2(pull(gpu, "THETA"), orc.theta))
        print(f"padded meta step {s}: " + " ".join(f"{k}={v:.2e}" for k, v in e.items()))
        assert e["gmeta"] < KTOL and e["glam_p"] < KTOL and e["h"] < TOL and e["theta"] < TOL
    # ---- invariants, GPU against itself
    (x, y), _ = _batches(wl, 5)
    lens = np.array([S, 7, 64, 1, 100], dtype=np.int32)

    def grad_of(xx, ll):
        push_state(orc, gpu)
        gpu.base_step(dev_batch(gpu, xx, y, lens=ll))
        return pull(gpu, "G").copy(), pull(gpu, "LOSSES")[:5].copy()
    g_none, l_none = grad_of(x, None)
    g_full, l_full = grad_of(x, np.full(5, S, dtype=np.int32))
    assert np.array_equal(g_none, g_full) and np.array_equal(l_none, l_full)
    g_a, l_a = grad_of(x, lens)
    x2 = x.copy()
    for b in range(5):
        x2[b, lens[b]:] = V - 1 - b
    g_b, l_b = grad_of(x2, lens)
    tok = orc.model.slices["tok_emb"][0]
    keep = np.ones(g_a.size, dtype=bool); keep[tok:tok + V * wl.dims[1]] = False
    assert np.array_equal(l_a, l_b) and np.array_equal(g_a[keep], g_b[keep])
    tg_a, tg_b = g_a[tok:tok + V * wl.dims[1]].reshape(V, -1), g_b[tok:tok + V * wl.dims[1]].reshape(V, -1)
    real = np.unique(np.concatenate([x[b, :lens[b]] for b in range(5)]))
    assert np.array_equal(tg_a[real], tg_b[real])
    assert np.all(tg_b[[V - 1 - b for b in range(1, 5) if (V - 1 - b) not in real]] == 0.0)      # pad-only tokens: no gradient
    # out-of-range lengths are clamped, not an error
    g_c, _ = grad_of(x, np.array([S + 50, 7, 64, 0, 100], dtype=np.int32))
    assert np.array_equal(g_c, g_a)
    gpu.close()


@pytest.mark.parametrize("S,padded,B", [(64, False, 3), (64, True, 5), (256, False, 3), (256, True, 3), (256, True, 32)])
def test_other_sequence_lengths(S, padded, B):
    """Sequence lengths 64 and 256 (the attention kernels are instantiated per length; 256 walks two tiles per wave):
    one base step and one meta step against the oracle, with and without padding.  The last case fills the 8192-token
    limit of a batch (32 sequences of 256)."""
    Bm = max(2, B // 2)
    wl = make_workload(3, n_train=8 * B, n_meta=8 * Bm, dims=(2, 128, 2, 256, S, 600, 3), batch=B, meta_batch=Bm)
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    lens = seq_lengths(wl.seed + S, 6 * B, S)
    lens[0], lens[1] = 1, S
    inp = (lambda x, l: with_lengths(x, l)) if padded else (lambda x, l: x)
    for s in range(3):
        (x, y), _ = _batches(wl, s)
        orc.base_step(inp(x, lens[B * (s + 1):B * (s + 2)]), y)
    (x, y), (xm, ym) = _batches(wl, 3)
    lt, lm = lens[:B], lens[5 * B:5 * B + Bm]
    push_state(orc, gpu)
    tb = dev_batch(gpu, x, y, lens=lt if padded else None)
    mb = dev_batch(gpu, xm, ym, lens=lm if padded else None)
    lo = orc.base_step(inp(x, lt), y)
    gpu.base_step(tb)
    g = pull(gpu, "G")
    errs = _group_errors(orc, g, orc.g)
    print(f"S={S} padded={padded} base: rel-L2 g {rel_l2(g, orc.g):.3e}; worst group {max(errs, key=errs.get)} {max(errs.values()):.3e}")
    assert rel_l2(g, orc.g) < KTOL and all(e < TOL for e in errs.values()), errs
    assert abs(float(pull(gpu, "SCALARS")[2]) - lo) < 2e-2 * abs(lo)
    push_state(orc, gpu)
    r = orc.meta_step(inp(x, lt), y, inp(xm, lm), ym)
    gpu.meta_step(tb, mb)
    e = dict(gmeta=rel_l2(pull(gpu, "GMETA"), r["g_meta"]), h=rel_l2(pull(gpu, "HYPERGRAD"), r["h"]),
             glam_p=rel_l2(pull(gpu, "GLAM_PLUS"), r["glam_p"]), theta=rel_l2(pull(gpu, "THETA"), orc.theta))
    print(f"S={S} padded={padded} meta: " + " ".join(f"{k}={v:.2e}" for k, v in e.items()))
    assert e["gmeta"] < KTOL and e["glam_p"] < KTOL and e["h"] < TOL and e["theta"] < TOL
    gpu.close()


@pytest.mark.parametrize("B,padded", [(32, False), (32, True), (33, False), (33, True)])
def test_attention_backward_on_both_sides_of_its_parts(B, padded):
    """256 heads of 128 positions take the backward pass in three parts, 264 in two: a base step against the oracle."""
    wl = make_workload(3, n_train=2 * B, n_meta=4, dims=(1, 512, 8, 512, 128, 600, 3), batch=B, meta_batch=2)
    orc, gpu = make_pair(wl, init_theta(wl, 0.05), init_lambda(wl), base_lr=1e-3)
    (x, y), _ = _batches(wl, 0)
    lens = seq_lengths(wl.seed + 7, B, 128)
    lens[:4] = 1, 128, 32, 33
    push_state(orc, gpu)
    orc.base_step(with_lengths(x, lens) if padded else x, y)
    gpu.base_step(dev_batch(gpu, x, y, lens=lens if padded else None))
    g = pull(gpu, "G")
    errs = _group_errors(orc, g, orc.g)
    print(f"B={B} padded={padded}: rel-L2 g {rel_l2(g, orc.g):.3e}; worst group {max(errs, key=errs.get)} {max(errs.values()):.3e}")
    assert rel_l2(g, orc.g) < KTOL and all(e < TOL for e in errs.values()), errs
    gpu.close()


def _golden_encoders():
    import importlib.util
    import json
    import os
    spec = importlib.util.spec_from_file_location("make_encoder_bits", os.path.join(os.path.dirname(__file__), "golden", "make_encoder_bits.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod, json.load(open(mod.FILE)) if os.path.exists(mod.FILE) else {}


GOLDEN, GOLDEN_BITS = _golden_encoders()


@pytest.mark.parametrize("case", GOLDEN.CASES, ids=GOLDEN.name_of)
def test_small_encoders_keep_their_bits(case):
    """Every output of a scored batch, a base and a meta step has the recorded bits: roundings and the order of sums have not changed anywhere on the way."""
    want, got = GOLDEN_BITS[GOLDEN.name_of(case)], GOLDEN.encoder_bits(case)
    assert got == want, {k: (got[k], want[k]) for k in want if got[k] != want[k]}


@pytest.mark.parametrize("S,padded", [(64, False), (64, True), (128, False), (128, True), (256, False), (256, True)])
def test_attention_with_scores_of_ten_to_the_twelfth(S, padded):
    """Wq = Wk = 2^17 I: every query takes its own key's value alone.  The largest score's weight is one however large it is, so logits and
    the gradients behind the scores are those of the oracle, and nothing is infinite.  (The scores' own gradients are differences that vanish.)"""
    dims = (1, 192, 3, 320, S, 300, 3)
    wl = make_workload(3, n_train=6, n_meta=2, dims=dims, batch=6, meta_batch=2)
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    off, shape = orc.model.slices["l0.Wqkv"]
    W = orc.theta[off:off + int(np.prod(shape))].reshape(shape)
    W[:192], W[192:384] = 2.0 ** 17 * np.eye(192), 2.0 ** 17 * np.eye(192)
    push_state(orc, gpu)
    x, y = wl.x_train[:6], wl.y_train[:6]
    lens = np.array([1, S, S // 2 + 3, 17, S - 1, 33], dtype=np.int32) if padded else None
    xo = with_lengths(x, lens) if padded else x
    import torch
    out = [torch.zeros(s, device=gpu.dev) for s in ((6, 3), (6,), (6,))]
    gpu.eval(dev_batch(gpu, x, y, lens=lens), *out)
    for got, want in zip(out, orc.evaluate(xo, y)):
        assert rel_l2(got.cpu().numpy(), want) < KTOL
    orc.base_step(xo, y)
    gpu.base_step(dev_batch(gpu, x, y, lens=lens))
    g = pull(gpu, "G")
    assert np.all(np.isfinite(g))
    errs = _group_errors(orc, g, orc.g)
    assert all(errs[k] < TOL for k in ("l0.Wo", "l0.W1", "l0.W2", "Wc")), errs
    gpu.close()


def test_out_of_range_ids_and_labels_are_clamped():
    """Token ids outside [0, V) and labels outside [0, C) are clamped on the device by every kernel that indexes with
    them (embedding gather, token-gradient scatter, per-sample stage): a batch carrying such values gives the bits of
    the batch with the clamped values, for the base step and for the meta step."""
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    V, C = wl.dims[5], wl.dims[6]
    (x, y), (xm, ym) = _batches(wl, 0)
    bad_x, bad_y = x.copy(), y.copy()
    bad_x[0, 3], bad_x[1, 7], bad_x[2, 0], bad_x[4, 127] = V + 5, -3, 2 ** 30, -2 ** 31
    bad_y[0], bad_y[3] = C + 2, -1
    res = []
    for xx, yy in ((bad_x, bad_y), (np.clip(bad_x, 0, V - 1), np.clip(bad_y, 0, C - 1))):
        _, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
        tb, mb = dev_batch(gpu, xx, yy), dev_batch(gpu, xm, ym)
        gpu.base_step(tb); gpu.base_step(tb); gpu.meta_step(tb, mb)
        res.append({k: pull(gpu, k).copy() for k in ("G", "THETA", "HYPERGRAD", "LAMBDA", "LOSSES")})
        assert np.all(np.isfinite(res[-1]["THETA"])) and int(pull(gpu, "COUNTERS")[2]) == 0
        gpu.close()
    for k in res[0]:
        assert np.array_equal(res[0][k], res[1][k]), k


@pytest.mark.usefixtures("backward_streams")
def test_non_finite_hypergradient_takes_back_the_early_nudge():
    """bf16 models nudge the GEMM block of theta in the pass that writes the +- halves, before the hypergradient exists.
    When the hypergradient then turns out not to be finite (a NaN planted in the weight net's output bias, which the
    direct-gradient pass never reads), the step is skipped like the oracle's: hypergradient 0, lambda and the meta
    moments untouched, the non-GEMM tail of theta untouched bit for bit, the GEMM block back at its old value up to one
    fp32 rounding -- and the working copy and its residual half follow, so the next base step gives the gradient of a
    context that never saw the skipped step."""
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    _, ref = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    for s in range(3):
        (x, y), (xm, ym) = _batches(wl, s)
        gpu.base_step(dev_batch(gpu, x, y)); ref.base_step(dev_batch(ref, x, y)); orc.base_step(x, y)
    lam = pull(gpu, "LAMBDA").copy(); lam_bad = lam.copy(); lam_bad[-1] = np.nan
    gpu.set_state("LAMBDA", lam_bad); orc.lam = lam_bad.astype(np.float64)
    th, mm = pull(gpu, "THETA").copy(), pull(gpu, "META_M").copy()
    r = orc.meta_step(x, y, xm, ym)
    assert orc.status == 1 and orc.meta_t == 0 and r["eps"] > 0
    gpu.meta_step(dev_batch(gpu, x, y), dev_batch(gpu, xm, ym))
    cnt = pull(gpu, "COUNTERS")
    assert int(cnt[1]) == 0 and int(cnt[2]) == 1 and float(pull(gpu, "SCALARS")[0]) > 0
    assert np.all(pull(gpu, "HYPERGRAD") == 0) and np.array_equal(pull(gpu, "META_M"), mm)
    assert np.array_equal(pull(gpu, "LAMBDA"), lam_bad, equal_nan=True)
    th2 = pull(gpu, "THETA")
    ng = _gemm_block(orc)
    assert np.array_equal(th2[ng:], th[ng:])
    assert np.max(np.abs(th2[:ng].astype(np.float64) - th[:ng])) <= 2.0 ** -23 * np.max(np.abs(th[:ng]))
    assert not np.array_equal(pull(gpu, "VDIR"), np.zeros_like(th))          # the direction itself was computed
    gpu.set_state("LAMBDA", lam)
    (x, y), _ = _batches(wl, 3)
    gpu.base_step(dev_batch(gpu, x, y)); ref.base_step(dev_batch(ref, x, y))
    assert rel_l2(pull(gpu, "G"), pull(ref, "G")) < 1e-4, rel_l2(pull(gpu, "G"), pull(ref, "G"))
    gpu.close(); ref.close()


def test_eval_small_encoder_with_padding():
    """sama_eval on the bf16 encoder, padded batch: logits, losses and weights against the oracle at the bf16 working
    weights (what the base step's forward sees)."""
    import torch
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    S = wl.dims[4]
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    (x, y), (xm, ym) = _batches(wl, 0)
    push_state(orc, gpu)
    orc.t = 1                                            # evaluate needs no history; keep the oracle's guard quiet
    lens = np.array([S, 9, 1, 77, 40], dtype=np.int32)
    zo = torch.zeros((5, wl.dims[-1]), device=gpu.dev); lo = torch.zeros(5, device=gpu.dev); wo = torch.zeros(5, device=gpu.dev)
    gpu.eval(dev_batch(gpu, x, y, lens=lens), zo, lo, wo)
    z, l, w = orc.evaluate(with_lengths(x, lens), y)
    print(f"eval: logits {rel_l2(zo.cpu().numpy(), z):.2e} losses {rel_l2(lo.cpu().numpy(), l):.2e} weights {rel_l2(wo.cpu().numpy(), w):.2e}")
    assert rel_l2(zo.cpu().numpy(), z) < KTOL and rel_l2(lo.cpu().numpy(), l) < KTOL and rel_l2(wo.cpu().numpy(), w) < KTOL
    gpu.close()


@pytest.mark.usefixtures("backward_streams")
def test_checkpoint_and_resume_continue_bit_for_bit():
    """The settable state (theta, the moments, the kept gradient, lambda and its moments, the counters) is everything a
    run needs: a fresh context that is handed the state of a run after 6 iterations continues with the bits of the
    uninterrupted run (bf16 encoder, one stream and two, scheduled rates)."""
    wl = make_workload(3, n_train=40, n_meta=12, **SMALL)
    names = ("THETA", "M", "V", "G", "LAMBDA", "META_M", "META_V")
    rate = lambda k: 1e-3 * (1.0 - 0.05 * k)

    def run(gpu, k0, k1):
        for k in range(k0, k1):
            (x, y), (xm, ym) = _batches(wl, k)
            tb, mb = dev_batch(gpu, x, y), dev_batch(gpu, xm, ym)
            gpu.set_lr(rate(k), 1e-3)
            gpu.base_step(tb); gpu.meta_step(tb, mb)

    _, a = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    run(a, 0, 6)
    saved = {n: pull(a, n).copy() for n in names}
    counters = pull(a, "COUNTERS").copy()
    run(a, 6, 10)
    want = {n: pull(a, n).copy() for n in names + ("HYPERGRAD", "COUNTERS")}
    a.close()
    _, b = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    for n in names:
        b.set_state(n, saved[n])
    b.set_state("COUNTERS", counters)
    run(b, 6, 10)
    for n in want:
        assert np.array_equal(pull(b, n), want[n]), n
    b.close()


@pytest.mark.usefixtures("backward_streams")
@pytest.mark.parametrize("d,heads,ffn", [(1280, 20, 1344), (2048, 32, 2048)])
def test_wide_encoder(d, heads, ffn):
    """Hidden widths above 1024 (the LayerNorm kernels then keep eight 16-byte pieces of a row per lane): one base step
    and one meta step against the oracle."""
    wl = make_workload(3, n_train=24, n_meta=8, dims=(1, d, heads, ffn, 64, 300, 3), batch=3, meta_batch=2)
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    for s in range(2):
        (x, y), _ = _batches(wl, s)
        orc.base_step(x, y)
    (x, y), (xm, ym) = _batches(wl, 2)
    push_state(orc, gpu)
    tb, mb = dev_batch(gpu, x, y), dev_batch(gpu, xm, ym)
    lo = orc.base_step(x, y)
    gpu.base_step(tb)
    g = pull(gpu, "G")
    errs = _group_errors(orc, g, orc.g)
    print(f"d={d} base: rel-L2 g {rel_l2(g, orc.g):.3e}; worst group {max(errs, key=errs.get)} {max(errs.values()):.3e}")
    assert rel_l2(g, orc.g) < KTOL and all(e < TOL for e in errs.values()), errs
    assert abs(float(pull(gpu, "SCALARS")[2]) - lo) < 2e-2 * abs(lo)
    push_state(orc, gpu)
    r = orc.meta_step(x, y, xm, ym)
    gpu.meta_step(tb, mb)
    e = dict(gmeta=rel_l2(pull(gpu, "GMETA"), r["g_meta"]), h=rel_l2(pull(gpu, "HYPERGRAD"), r["h"]),
             glam_p=rel_l2(pull(gpu, "GLAM_PLUS"), r["glam_p"]), theta=rel_l2(pull(gpu, "THETA"), orc.theta))
    e["glam_m"] = rel_l2(pull(gpu, "GLAM_MINUS"), r["glam_m"]); e["eps"] = abs(pull(gpu, "SCALARS")[0] - r["eps"]) / r["eps"]
    # h = -(g+ - g-) / (2 eps): with |dg+-| <= GBAR |g+-| and the relative error of eps <= EBAR, the relative error of h is
    # at most GBAR (|g+| + |g-|) / |g+ - g-| + EBAR -- a bar made of the oracle's numbers and the two fixed bars alone.
    # On this single-layer wide model at its initial point the two passes differ in the fourth digit only, so the
    # bar on h is far above the workloads' 2e-2; the inputs of the difference carry the tight bars.
    GBAR, EBAR = 2e-4, KTOL
    amplification = (np.linalg.norm(r["glam_p"]) + np.linalg.norm(r["glam_m"])) / np.linalg.norm(r["glam_p"] - r["glam_m"])
    hbar = GBAR * amplification + EBAR
    print(f"d={d} meta: " + " ".join(f"{k}={v:.2e}" for k, v in e.items()) + f" amplification={amplification:.1e} hbar={hbar:.2e}")
    assert e["gmeta"] < KTOL and e["theta"] < TOL
    assert e["glam_p"] < GBAR and e["glam_m"] < GBAR and e["eps"] < EBAR
    assert e["h"] < hbar
    gpu.close()


@pytest.mark.parametrize("d,B,lens,repeat", [
    (192, 1, [1], False), (192, 1, [16], False), (192, 2, [17, 128], False), (192, 5, [1, 15, 16, 113, 128], True),
    (192, 5, [1, 1, 1, 1, 1], True), (320, 9, None, True), (320, 6, None, False)])
def test_padded_rows_and_embedding_gradients_at_their_edges(d, B, lens, repeat):
    """Base step against the oracle where the packing of padded rows can go wrong (lengths beside the 16-row groups, one token in
    all) and where the embedding gradients can (one token id at every position, 1152 rows of one sum; batches that are no multiple
    of the four sequences whose rows fill a tile of the last layer)."""
    S = 128
    wl = make_workload(3, n_train=4 * B, n_meta=4, dims=(2, d, d // 64, 320, S, 600, 3), batch=B, meta_batch=2)
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    (x, y), _ = _batches(wl, 0)
    if repeat:
        x = np.full_like(x, 7)
    xo = x if lens is None else with_lengths(x, np.array(lens, dtype=np.int32))
    push_state(orc, gpu)
    lo = orc.base_step(xo, y)
    gpu.base_step(dev_batch(gpu, x, y, lens=None if lens is None else np.array(lens, dtype=np.int32)))
    g = pull(gpu, "G")
    print(f"d={d} B={B} lens={lens}: rel-L2 g {rel_l2(g, orc.g):.3e}")
    assert rel_l2(g, orc.g) < KTOL
    for name in ("tok_emb", "pos_emb", "Wc", "bc"):
        off, shape = orc.model.slices[name]
        sl = slice(off, off + int(np.prod(shape)))
        assert rel_l2(g[sl], orc.g[sl]) < TOL, name
    assert abs(float(pull(gpu, "SCALARS")[2]) - lo) < 2e-2 * abs(lo)
    gpu.close()


@pytest.mark.parametrize("d,counts", [(256, (1, 8, 9, 64, 65, 130)), (320, (1, 8, 9, 64, 65, 130))])
def test_embedding_gradients_of_repeated_ids(d, counts):
    """Ids that occur as often as their rows are fetched together, one less and one more, first seen among the positions whose
    columns go to a workgroup each (the first 512) and behind them.  The sum of a token's rows is a sum over rows of 2 layers' output
    gradient, so its error is that of the pass.  A missing or doubled row could hide in that, so all tokens' sums are added up and
    compared with the positions' sums, which add the same rows: the two differ by fp32 roundings of B S summands."""
    S, B = 128, 9
    wl = make_workload(3, n_train=4 * B, n_meta=4, dims=(2, d, d // 64, 320, S, 1400, 3), batch=B, meta_batch=2)
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    (x, y), _ = _batches(wl, 0)
    flat = np.arange(100, 100 + B * S).astype(x.dtype)     # every position its own id
    rng = np.random.default_rng(5)
    early = rng.permutation(np.arange(20, 512)); late = rng.permutation(np.arange(530, B * S))
    e = l = 0
    for k, n in enumerate(counts):
        flat[early[e:e + (n + 1) // 2]] = k; flat[late[l:l + n // 2]] = k; e += (n + 1) // 2; l += n // 2      # first seen early
        flat[late[l:l + n]] = 50 + k; l += n                                                                # first seen late
    x = flat.reshape(B, S)
    push_state(orc, gpu)
    orc.base_step(x, y)
    gpu.base_step(dev_batch(gpu, x, y))
    off, shape = orc.model.slices["tok_emb"]
    got, want = pull(gpu, "G")[off:off + int(np.prod(shape))].reshape(shape), orc.g[off:off + int(np.prod(shape))].reshape(shape)
    for k in [i for i in range(len(counts))] + [50 + i for i in range(len(counts))]:
        assert np.count_nonzero(x == k) == counts[k % 50]
        assert rel_l2(got[k], want[k]) < TOL, (k, rel_l2(got[k], want[k]))
    assert rel_l2(got, want) < KTOL
    # the gradients of the positions' rows, of which every token's is a sum: pos_emb sums them over the sequences
    po, ps = orc.model.slices["pos_emb"]
    assert np.allclose(pull(gpu, "G")[po:po + int(np.prod(ps))].reshape(ps).sum(0, dtype=np.float64), got.sum(0, dtype=np.float64),
                       rtol=0, atol=B * S * 2.0 ** -24 * np.abs(got).sum(0).max())
    gpu.close()


@pytest.mark.parametrize("d,ffn,S,B,padded", [
    (128, 256, 64, 1, False), (192, 448, 64, 2, True), (192, 448, 128, 1, False), (320, 1088, 128, 1, True), (192, 384, 128, 8, False),
    (192, 448, 128, 9, True)])
def test_eval_of_few_rows(d, ffn, S, B, padded):
    """sama_eval of one text, of two short ones, and of a few (whose last layer keeps 128 or 192 rows), against the oracle: the
    smallest tiles, contractions of fewer and of more slabs than those have in flight."""
    import torch
    wl = make_workload(3, n_train=4 * B, n_meta=4, dims=(2, d, d // 64, ffn, S, 600, 3), batch=B, meta_batch=2)
    orc, gpu = make_pair(wl, init_theta(wl, 0.05), init_lambda(wl), base_lr=1e-3)
    (x, y), _ = _batches(wl, 0)
    push_state(orc, gpu)
    orc.t = 1
    lens = np.minimum(S, 1 + 37 * np.arange(1, B + 1)).astype(np.int32)
    out = [torch.zeros(s, device=gpu.dev) for s in ((B, 3), (B,), (B,))]
    gpu.eval(dev_batch(gpu, x, y, lens=lens if padded else None), *out)
    for name, got, want in zip(("logits", "losses", "weights"), out, orc.evaluate(with_lengths(x, lens) if padded else x, y)):
        print(f"{name} {rel_l2(got.cpu().numpy(), want):.2e}")
        assert rel_l2(got.cpu().numpy(), want) < KTOL
    gpu.close()


@pytest.mark.parametrize("S,fast,padded", [(128, 0, False), (128, 0, True), (128, 1, False), (64, 0, True)])
def test_eval_of_a_text_does_not_depend_on_what_is_scored_beside_it(S, fast, padded):
    """sama_eval of each text alone, of the whole batch, and the base step's own losses on that batch: the same bits.  One text
    has few rows and takes other tiles than the batch does; every sum keeps its order."""
    import torch
    B = 5
    wl = make_workload(3, n_train=4 * B, n_meta=4, dims=(3, 192, 3, 448, S, 600, 3), batch=B, meta_batch=2)
    orc, gpu = make_pair(wl, init_theta(wl, 0.05), init_lambda(wl), base_lr=1e-3, fast_base_pass=fast)
    (x, y), _ = _batches(wl, 0)
    lens = np.minimum(S, 1 + 29 * np.arange(1, B + 1)).astype(np.int32) if padded else None

    def score(sel):
        out = [torch.zeros(s, device=gpu.dev) for s in ((len(sel), 3), (len(sel),), (len(sel),))]
        gpu.eval(dev_batch(gpu, x[sel], y[sel], lens=None if lens is None else lens[sel]), *out)
        return [o.cpu().numpy() for o in out]
    every = score(np.arange(B))
    for i in range(B):
        for name, one, all_ in zip(("logits", "losses", "weights"), score(np.array([i])), every):
            assert np.array_equal(one[0], all_[i]), (name, i)
    gpu.base_step(dev_batch(gpu, x, y, lens=lens))
    assert np.array_equal(pull(gpu, "LOSSES")[:B], every[1])
    gpu.close()


@pytest.mark.parametrize("B,padded", [(2, False), (3, True)])
def test_weights_fetched_ahead(B, padded):
    """16 million weights of 8 layers, with their state more than the last-level cache holds, and few rows: the LayerNorms' launches
    fetch the next weights beside their rows.  A base step and the passes of a meta step against the oracle."""
    wl = make_workload(3, n_train=2 * B, n_meta=4, dims=(8, 448, 7, 1344, 64, 300, 3), batch=B, meta_batch=2)
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    (x, y), (xm, ym) = _batches(wl, 0)
    lens = np.array([1, 64, 33][:B], dtype=np.int32) if padded else None
    xo = with_lengths(x, lens) if padded else x
    for _ in range(3):   # after a single one every entry of Eq. 4's direction is the sign of its gradient, which rounding decides
        orc.base_step(xo, y)
    push_state(orc, gpu)
    orc.base_step(xo, y)
    gpu.base_step(dev_batch(gpu, x, y, lens=lens))
    g = pull(gpu, "G")
    errs = _group_errors(orc, g, orc.g)
    print(f"B={B} padded={padded}: rel-L2 g {rel_l2(g, orc.g):.3e}; worst group {max(errs, key=errs.get)} {max(errs.values()):.3e}")
    assert rel_l2(g, orc.g) < KTOL and all(e < TOL for e in errs.values()), errs
    push_state(orc, gpu)
    r = orc.meta_step(xo, y, xm, ym)
    gpu.meta_step(dev_batch(gpu, x, y, lens=lens), dev_batch(gpu, xm, ym))
    e = dict(gmeta=rel_l2(pull(gpu, "GMETA"), r["g_meta"]), glam_p=rel_l2(pull(gpu, "GLAM_PLUS"), r["glam_p"]))
    print(" ".join(f"{k}={v:.2e}" for k, v in e.items()))
    assert e["gmeta"] < KTOL and e["glam_p"] < KTOL
    gpu.close()


@pytest.mark.parametrize("B,dims,kept", [(60, (4, 640, 10, 1280), 52), (60, (4, 640, 10, 1280), 100), (60, (4, 640, 10, 1280), 124), (36, (2, 1024, 16, 4096), 52),
                                         (36, (2, 1024, 16, 4096), 100), (36, (2, 1024, 16, 4096), 124)])
def test_weights_fetched_ahead_of_many_padded_rows(B, dims, kept):
    """7680 rows of 640 with about 3100, 6000 and 7400 in use, 4608 of 1024 with 2000, 3700 and 4500: the LayerNorms of a base step fetch the next
    weights with the first two of each.  Scoring never does at these sizes; the losses of both are the same bits."""
    import torch
    wl = make_workload(3, n_train=B, n_meta=2, dims=dims + (128, 300, 3), batch=B, meta_batch=2)
    _, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    x, y = wl.x_train[:B], wl.y_train[:B]
    lens = np.clip(np.arange(B) % 9 - 4 + kept, 1, 128).astype(np.int32)
    out = [torch.zeros(s, device=gpu.dev) for s in ((B, 3), (B,), (B,))]
    gpu.eval(dev_batch(gpu, x, y, lens=lens), *out)
    gpu.base_step(dev_batch(gpu, x, y, lens=lens))
    assert np.isfinite(pull(gpu, "G")).all()
    assert np.array_equal(pull(gpu, "LOSSES")[:B], out[1].cpu().numpy())
    gpu.close()


@pytest.mark.parametrize("B,dims,S,padded", [(88, (3, 192, 3, 320), 64, False), (90, (3, 192, 3, 320), 64, True), (30, (3, 320, 5, 640), 128, False), (29, (4, 320, 5, 640), 128, True),
                                             (13, (3, 704, 11, 1408), 128, True), (8, (3, 1024, 16, 1024), 128, False), (9, (3, 1024, 16, 1024), 128, False), (48, (3, 192, 3, 320), 64, True), (10, (3, 640, 10, 1280), 128, False), (32, (3, 1024, 16, 2048), 256, False), (33, (2, 640, 10, 1280), 64, True)])
def test_residual_made_from_the_layernorms_input(B, dims, S, padded):
    """From 2^20 elements of rows x width on the products make the residual themselves, below it the LayerNorm stores it: texts scored alone and in such a batch have the same bits.
    8 sequences of 1024 are exactly that many; 48 of 192 and 10 of 640 have more than half, so that a pass stores it and the two stacked ones of a meta step make it.
    Widths with tiles cut short, any number of rows in use.
    The stacked passes, whose gains and shifts are perturbed, against the oracle."""
    import torch
    C, d = 3, dims[1]
    wl = make_workload(3, n_train=B, n_meta=2, dims=dims + (S, 300, C), batch=B, meta_batch=2)
    orc, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    x, y = wl.x_train[:B], wl.y_train[:B]
    lens = np.clip((np.arange(B) * 37) % (2 * S), 1, S).astype(np.int32) if padded else None

    def score(sel):
        out = [torch.zeros(s, device=gpu.dev) for s in ((len(sel), C), (len(sel),), (len(sel),))]
        gpu.eval(dev_batch(gpu, x[sel], y[sel], lens=None if lens is None else lens[sel]), *out)
        return [o.cpu().numpy() for o in out]
    push_state(orc, gpu)
    every = score(np.arange(B))
    for i in (0, 1, B // 2, B - 1):
        for name, one, all_ in zip(("logits", "losses", "weights"), score(np.array([i])), every):
            assert np.array_equal(one[0], all_[i]), (name, i)
    gpu.base_step(dev_batch(gpu, x, y, lens=lens))
    assert np.array_equal(pull(gpu, "LOSSES")[:B], every[1])
    if B * S * d < 1500000:   # the oracle's time
        xo = with_lengths(x, lens) if padded else x
        for _ in range(3):
            orc.base_step(xo, y)
        push_state(orc, gpu)
        orc.base_step(xo, y)
        gpu.base_step(dev_batch(gpu, x, y, lens=lens))
        errs = _group_errors(orc, pull(gpu, "G"), orc.g)
        assert rel_l2(pull(gpu, "G"), orc.g) < KTOL and all(e < TOL for e in errs.values()), errs
        push_state(orc, gpu)
        r = orc.meta_step(xo, y, wl.x_meta[:2], wl.y_meta[:2])
        gpu.meta_step(dev_batch(gpu, x, y, lens=lens), dev_batch(gpu, wl.x_meta[:2], wl.y_meta[:2]))
        e = dict(gmeta=rel_l2(pull(gpu, "GMETA"), r["g_meta"]), glam_p=rel_l2(pull(gpu, "GLAM_PLUS"), r["glam_p"]), glam_m=rel_l2(pull(gpu, "GLAM_MINUS"), r["glam_m"]))
        print(" ".join(f"{k}={v:.2e}" for k, v in e.items()))
        assert all(v < KTOL for v in e.values()), e
    gpu.close()


@pytest.mark.parametrize("C,d", [(8, 192), (9, 192), (21, 1088)])
def test_head_of_many_classes_and_features(C, d):
    """The classifier with as many classes as are taken at a time, one more, and three times as many over more features than are:
    a text alone (a wave) and among eleven others (two samples to a wave), bit for bit; the logits against the oracle."""
    import torch
    wl = make_workload(3, n_train=12, n_meta=2, dims=(1, d, d // 64, 128, 64, 300, C), batch=12, meta_batch=2)
    orc, gpu = make_pair(wl, init_theta(wl, 0.05), init_lambda(wl), base_lr=1e-3)
    x, y = wl.x_train[:12], wl.y_train[:12]
    push_state(orc, gpu)
    out = [[torch.zeros(s, device=gpu.dev) for s in ((n, C), (n,), (n,))] for n in (12, 1)]
    gpu.eval(dev_batch(gpu, x, y), *out[0])
    gpu.eval(dev_batch(gpu, x[:1], y[:1]), *out[1])
    for all_, one in zip(*out):
        assert torch.equal(all_[:1], one)
    assert rel_l2(out[0][0].cpu().numpy(), orc.evaluate(x, y)[0]) < KTOL
    gpu.close()


def _rows_counts(L):
    """Launches of the kernel that chooses its tile on the device since the last call: forward, input gradients."""
    import ctypes
    c = (ctypes.c_int64 * 2)()
    assert L.sama_dev_gemm_counts(c, ctypes.c_int32(2)) == 0
    return list(c)


ROWS_CHOICES = [0] + [int(k * 16, 16) for k in "1245"] + [0x1245544221145512]   # the heuristic's, one tile for all, a mixture


@pytest.mark.parametrize("dims", [(2, 320, 5, 896, 128, 300, 3), (2, 768, 12, 1536, 64, 300, 2), (2, 768, 12, 3072, 128, 300, 2)])
def test_tile_chosen_by_the_rows_in_use(dims):
    """Padded batches with from an eighth to all of their rows in use, at widths that leave ragged tiles and whole ones: with the tile
    chosen on the device by the rows, as the heuristic does and each of the four for each product (forward, paired and input gradients, all epilogues),
    every bit of a base step and of a meta step is that of one tile for all of them."""
    import ctypes
    from paper_2310_05674_amd import binding as B
    L = B.load_library()
    S, n = dims[4], 4096 // dims[4]
    wl = make_workload(3, n_train=2 * n, n_meta=8, dims=dims, batch=n, meta_batch=4)
    _, gpu = make_pair(wl, init_theta(wl, 0.02), init_lambda(wl), base_lr=1e-3)
    (x, y), (xm, ym) = _batches(wl, 0)
    start = {k: pull(gpu, k).copy() for k in ("THETA", "M", "V", "G", "LAMBDA", "META_M", "META_V")}
    r = np.random.default_rng(5)
    lens_sets = [np.full(n, k, dtype=np.int32) for k in sorted({1, 16, 17, S // 4 + 1, S // 2, S // 2 + 1, 3 * S // 4, S - 17, S - 16, S})]
    lens_sets += [r.integers(1, S + 1, n).astype(np.int32) for _ in range(3)]
    products = 4 * dims[0]                       # of a pass; the last layer's rows behind its attention are not those in use
    taken = [0, 0]

    def step(lens, shape, choice):
        L.sama_dev_gemm_shape(ctypes.c_int32(shape))
        assert L.sama_dev_gemm_rows(ctypes.c_uint64(choice)) == 0
        for k, v in start.items():
            gpu.set_state(k, v)
        gpu.set_state("COUNTERS", np.array([3, 1, 0, 0], dtype=np.int64))
        tb = dev_batch(gpu, x, y, lens=lens)
        gpu.base_step(tb); gpu.meta_step(tb, dev_batch(gpu, xm, ym, lens=lens[:4]))
        return [pull(gpu, k) for k in ("G", "THETA", "GMETA", "HYPERGRAD")]
    try:
        for lens in lens_sets:
            want = step(lens, 15, 0)
            assert all(np.isfinite(a).all() for a in want)
            _rows_counts(L)
            for choice in ROWS_CHOICES:
                got = step(lens, 0, choice)
                assert all(np.array_equal(a, b) for a, b in zip(got, want)), (hex(choice), int(lens.sum()), lens[:4])
                c = _rows_counts(L)
                if choice == 0:
                    taken = [a + b for a, b in zip(taken, c)]
                else:                            # two backward passes; their forward passes and the stacked one
                    assert c[0] == 3 * (products - 3) and c[1] == 2 * (products - 3), c
        assert taken[0] > 0 and (taken[1] > 0 or dims[1] == 320), taken   # the heuristic does choose this launch
    finally:
        L.sama_dev_gemm_shape(ctypes.c_int32(0)); L.sama_dev_gemm_rows(ctypes.c_uint64(0))
        gpu.close()
