"""The per-cell kernels at the edges of a wave: the mixture step's feature counts, the evaluation head's batches
and neighbourhoods (one launch with the fitness up to seven individuals and 64 rows,
two beyond)."""
import numpy as np
import pytest
from test_gpu_parity import _close, _setup, _warm_state

from oracle import coevo, mixture

torch = pytest.importorskip("torch")
from harness import GpuGrid, check_mixture, fp32_state  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("features", [1, 63, 64, 65, 130])
def test_mixture_matches_oracle_at_any_feature_count(features):
    wl, data, _ = _setup("ragged_2x3")
    wl = dict(wl, mix_enable=1, mix_samples=77, mix_feat_dim=features)
    S = coevo.Setup(wl, len(data))
    st = _warm_state(S, data, steps=1)
    g0 = np.random.default_rng(1)
    st.w = fp32_state(coevo.State(**{**{f: getattr(st, f) for f in coevo.State.FIELDS},
                                     "w": g0.dirichlet(np.ones(5), size=S.C)})).w
    stats = mixture.real_stats(S, data)
    print(f"[case] mixture features={features}", flush=True)
    with GpuGrid(wl, data) as gg:
        gg.set_state(st)
        w, sc, acc = gg.mixture(0)
        check_mixture(S, st, stats, 0, w, sc, acc)


@pytest.mark.parametrize("batch,pop,mode", [(1, 1, 0), (63, 1, 1), (64, 1, 0), (65, 1, 1), (3, 2, 1)])
def test_eval_matches_oracle_at_any_batch(batch, pop, mode):
    wl, data, _ = _setup("ragged_2x3")
    wl = dict(wl, batch=batch, pop_size=pop, fitness_mode=mode)
    S = coevo.Setup(wl, len(data))
    st = _warm_state(S, data, steps=1)
    print(f"[case] eval batch={batch} pop={pop} mode={mode}", flush=True)
    with GpuGrid(wl, data) as gg:
        gg.set_state(st)
        for a, b in zip(gg.eval(1), coevo.evaluate(S, st, data, 1)):
            assert _close(a, b, wl), np.max(np.abs(a - b) / np.abs(b))


@pytest.mark.parametrize("image_channels,g_hidden,d_hidden", [(1, [36, 20], [20, 36]), (4, [132, 12], [12, 132])])
def test_dcgan_with_channels_off_every_power_of_two(image_channels, g_hidden, d_hidden, monkeypatch):
    """Batch norm's and the patch kernels' walks over channels that do not divide their strides."""
    import test_gpu_dcgan as dc

    wl = dc._wl(rows=2, cols=2, img=(16, 16, image_channels), x_dim=256 * image_channels, z_dim=8, g_hidden=g_hidden,
                d_hidden=d_hidden, batch=5, lr0_g=2e-3, lr0_d=2e-3,
                data=dict(dc.WORKLOADS["dc16_2x2"]()["data"], c=image_channels, n=500 + image_channels))
    monkeypatch.setitem(dc.WORKLOADS, "odd", lambda: wl)
    dc.test_eval_matches_oracle("odd")
    dc.test_train_step_matches_oracle("odd", 1)


def test_evaluation_with_split_weights_leaves_training_alone():
    """A DCGAN grid large enough that the evaluation splits its weights ahead (into the idle gradient partials): the
    evaluation repeats bit for bit after a training step's partials went there, and the step's results are those of a
    step without an evaluation before it."""
    import synth

    wl = synth.small_workload("celeba_dcgan_4x4", rows=2, cols=2, img=(64, 64, 3), x_dim=64 * 64 * 3, z_dim=16,
                              g_hidden=[256, 128, 64, 32], d_hidden=[32, 64, 128, 256], batch=16,
                              data=dict(n=256, h=64, w=64))
    data = synth.make_dataset(wl["data"])
    print("[case] dcgan 64x64 eval around a training step", flush=True)
    with GpuGrid(wl, data) as a, GpuGrid(wl, data) as b:
        first = a.eval(0)
        st = a.get_state()
        la, lb = a.train(0, 0, 1), b.train(0, 0, 1)
        assert np.array_equal(la, lb)
        sa, sb = a.get_state(), b.get_state()
        for f in ("Gp", "Gm", "Gv", "Dp", "Dm", "Dv"):
            assert np.array_equal(getattr(sa, f), getattr(sb, f)), f
        a.set_state(st)
        for x, y in zip(a.eval(0), first):
            assert np.array_equal(x, y)
