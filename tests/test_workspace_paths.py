"""Workspace sizes on the CPU: a buffer sized for a range of cache tokens
serves every shorter range (chunked compaction shares one), whatever the
number of key splits each length takes."""
import dataclasses

import pytest

from paper_2606_07878_amd import binding, configs


@pytest.mark.parametrize("wid,mode", [(1, 0), (2, 0), (5, 0), (2, 1)])
@pytest.mark.parametrize("t", [1, 64, 65, 333, 1024])
def test_workspace_does_not_shrink_with_more_tokens(wid, mode, t):
    c = binding.make_config(configs.get_workload(wid).cfg, mode)
    sizes = [binding.still_workspace_size(c, n, t, 1) for n in list(range(1, 4200, 37)) + [5003, 8192, 9216, 20000, 65536]]
    assert sizes[0] > 0
    assert sizes == sorted(sizes)


def _size(cfg, N, t, mode=configs.MODE_BF16, **changes):
    return binding.still_workspace_size(binding.make_config(dataclasses.replace(cfg, **changes), mode), N, t, 1)


@pytest.mark.parametrize("wid,N,t,gb", [(2, 8192, 256, 2.8), (2, 8192, 1024, 3.1), (2, 5003, 333, 2.4),
                                        (2, 65536, 64, 10.3), (5, 9216, 1024, 5.6)])
def test_candidate_lists_stay_small(wid, N, t, gb):
    """The lists of a latent hold about 1536 entries over its key splits,
    however the splits are chosen (once 8 x 512 per split: 5.96, 4.38, 5.47,
    11.8 and 6.83 GB here)."""
    assert _size(configs.get_workload(wid).cfg, N, t) <= gb * 1e9


@pytest.mark.parametrize("mode,gb", [(configs.MODE_BF16, 0.3), (configs.MODE_FP32, 0.4)])
def test_no_refinement_buffers_without_refinement(mode, gb):
    """The two-block compactor of width 256 at logits scaled by 1/16 recomputes
    no logits and reserves nothing for it (4.6 and 2.1 GB otherwise)."""
    cfg = dataclasses.replace(configs.get_workload(2).cfg, latent_dim=256, n_blocks=2, cross_every_block=1,
                              n_cross_heads=1, n_self_heads=1, ffn_kind=configs.FFN_NONE, ffn_hidden=0)
    assert _size(cfg, 8192, 1024, mode, logit_scale_cross=1 / 16) <= gb * 1e9
    assert _size(cfg, 8192, 1024, mode, logit_scale_cross=1.0) > 3 * gb * 1e9 / 1.2


@pytest.mark.parametrize("mode", [configs.MODE_BF16, configs.MODE_FP32])
def test_refinement_rule_takes_the_magnitude_of_the_scale(mode):
    cfg = configs.get_workload(1).cfg
    assert (_size(cfg, 2048, 256, mode, logit_scale_cross=-1024.0) == _size(cfg, 2048, 256, mode, logit_scale_cross=1024.0)
            > _size(cfg, 2048, 256, mode, logit_scale_cross=-0.1) == _size(cfg, 2048, 256, mode, logit_scale_cross=0.1))


@pytest.mark.parametrize("mode", [configs.MODE_BF16, configs.MODE_FP32])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("group,nq", [(1, 1), (2, 1), (3, 1), (2, 2), (4, 2), (4, 4), (4, 8)])
def test_attention_workspace_does_not_shrink_with_more_keys(group, nq, d, mode):
    """Consumer attention: a buffer sized for a context serves every shorter
    one, past the number of chunks that one launch holds and on both sides of
    the choice between its kernels."""
    for H in (1, 8, 40):
        for t in (0, 655):
            lens = sorted({*range(33, 20000, 241), *(12288 // H + x - t for x in (-1, 0, 1) if 12288 // H > t + 32),
                           8192, 8200, 8256, 16384, 16392, 65536, 131072, 131080})
            sizes = [binding.still_attend_workspace_size(binding.still_attend_config(H, group, d, nq, t, S, 0, 0.0, mode, 0.0))
                     for S in lens]
            assert sizes[0] > 0
            assert sizes == sorted(sizes)
