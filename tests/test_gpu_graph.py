"""A whole iteration (base step + meta step) captured into a HIP graph and replayed: every replay must give the bits of
the same calls made eagerly, with new batch contents copied into the captured buffers between replays and the
program's own eager work and synchronisations in between.  The step-dependent optimizer scalars live on the device,
so a replay continues the step count where the previous one stopped."""
import numpy as np
import pytest
from datagen import make_workload, init_theta, init_lambda

pytestmark = pytest.mark.gpu


def _run(cfg, small=None, replays=4):
    import torch
    import paper_2310_05674_amd as pkg
    wl = make_workload(cfg, **(small or {}))
    th0, lam0 = init_theta(wl), init_lambda(wl)
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)               # capture needs a stream other than the default one
    kw = dict(H=wl.H, max_batch=wl.batch, max_meta_batch=wl.meta_batch, base_lr=wl.base_lr, meta_lr=wl.meta_lr, alpha=wl.alpha)

    def batches(k):
        it, im = wl.train_batch(k), wl.meta_batch_idx(k)
        return (np.ascontiguousarray(wl.x_train[it]), wl.y_train[it].astype(np.int32),
                np.ascontiguousarray(wl.x_meta[im]), wl.y_meta[im].astype(np.int32))

    with torch.cuda.stream(stream):
        eager = pkg.Sama(pkg.SamaConfig.make(wl.kind, wl.dims, **kw), th0, lam0)
        graph = pkg.Sama(pkg.SamaConfig.make(wl.kind, wl.dims, **kw), th0, lam0)
        x, y, xm, ym = (torch.as_tensor(a, device=dev) for a in batches(0))
        out = {}
        for s in (eager, graph):                          # one eager iteration each: lazy set-up happens outside the capture
            tb, mb = s.batch(x, y), s.batch(xm, ym)
            s.base_step(tb); s.meta_step(tb, mb)
            out[s] = (tb, mb)
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
            graph.base_step(out[graph][0]); graph.meta_step(*out[graph])
        # the capture itself executes nothing: bring the eager context level with it
        for k in range(1, replays + 1):
            bx, by, bxm, bym = batches(k)
            x.copy_(torch.as_tensor(bx)); y.copy_(torch.as_tensor(by)); xm.copy_(torch.as_tensor(bxm)); ym.copy_(torch.as_tensor(bym))
            g.replay()
            eager.base_step(out[eager][0]); eager.meta_step(*out[eager])
            stream.synchronize()
            for name in ("THETA", "LAMBDA", "M", "V", "HYPERGRAD", "COUNTERS"):
                a, b = graph.get_state(name).cpu().numpy(), eager.get_state(name).cpu().numpy()
                assert np.array_equal(a, b), (k, name)
            cnt = graph.get_state("COUNTERS").cpu().numpy()
            assert int(cnt[0]) == 1 + k and int(cnt[1]) == 1 + k and int(cnt[2]) == 0
        # eager calls and replays interleaved on one context (every pass that writes theta keeps the residual half of the
        # split weights current, so neither kind of call depends on which kind ran before it)
        bx, by, bxm, bym = batches(replays + 1)
        x.copy_(torch.as_tensor(bx)); y.copy_(torch.as_tensor(by)); xm.copy_(torch.as_tensor(bxm)); ym.copy_(torch.as_tensor(bym))
        graph.base_step(out[graph][0]); eager.base_step(out[eager][0])
        g.replay()
        eager.base_step(out[eager][0]); eager.meta_step(*out[eager])
        graph.meta_grad(*out[graph]); eager.meta_grad(*out[eager])
        stream.synchronize()
        assert np.array_equal(graph.get_state("HYPERGRAD").cpu().numpy(), eager.get_state("HYPERGRAD").cpu().numpy())
        graph.meta_step(*out[graph]); eager.meta_step(*out[eager])
        stream.synchronize()
        for name in ("THETA", "LAMBDA", "M", "V", "HYPERGRAD", "COUNTERS"):
            assert np.array_equal(graph.get_state(name).cpu().numpy(), eager.get_state(name).cpu().numpy()), ("interleaved", name)
        eager.close(); graph.close()


def test_graph_replay_mlp():
    _run(2)


@pytest.mark.usefixtures("backward_streams")
def test_graph_replay_small_encoder():
    _run(3, dict(n_train=40, n_meta=12, dims=(2, 192, 3, 320, 128, 600, 3), batch=5, meta_batch=3))
