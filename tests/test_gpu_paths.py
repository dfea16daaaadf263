"""GPU parity at the edges of the launch rules: sizes and options on both sides
of each choice between kernels, against the fp64 oracle."""
import pytest

from paper_2606_07878_amd import configs, synth
from tests.helpers import BF16_TOL, FP32_TOL, assert_parity, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _layer_case(w, mode, N, t, name):
    w = configs.shrink(w, n_tokens=N, t=t)
    cache, wts = synth.make_cache(w, 0), synth.make_weights(w, 0)
    ref = run_oracle(w.cfg, cache, wts, w.rope_theta, t)
    got = run_gpu(w.cfg, cache, wts, w.rope_theta, t, mode=mode)
    assert_parity(got, ref, BF16_TOL if mode == configs.MODE_BF16 else FP32_TOL, name)


@pytest.mark.parametrize("mode", [configs.MODE_BF16, configs.MODE_FP32])
@pytest.mark.parametrize("scale", [0.173, 0.174])
def test_refinement_rule_edge(mode, scale):
    """Logit scales just below and just above the one (log2 e times it = 1/4)
    from which the near-maximal logits are recomputed."""
    w = configs.shrink(configs.get_workload(1), logit_scale_cross=scale)
    _layer_case(w, mode, 1000, 130, f"cfg1 scale {scale} mode {mode}")
