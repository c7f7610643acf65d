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
