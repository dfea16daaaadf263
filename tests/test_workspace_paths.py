"""Workspace sizes on the CPU: a buffer sized for a range of cache tokens
serves every shorter range (chunked compaction shares one), whatever the
number of key splits each length takes."""
import pytest

from paper_2606_07878_amd import binding, configs


@pytest.mark.parametrize("wid,mode", [(1, 0), (2, 0), (5, 0), (2, 1)])
@pytest.mark.parametrize("t", [1, 64, 65, 333, 1024])
def test_workspace_does_not_shrink_with_more_tokens(wid, mode, t):
    c = binding.make_config(configs.get_workload(wid).cfg, mode)
    sizes = [binding.still_workspace_size(c, n, t, 1) for n in list(range(1, 4200, 37)) + [5003, 8192, 9216, 20000, 65536]]
    assert sizes[0] > 0
    assert sizes == sorted(sizes)
