"""Host logic of the tuner (no GPU): each lanes-per-query candidate is timed
as a launch of its own."""
import pytest

from paper_2206_13574_amd import tune
from tests import fake_hip


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    return fake_hip.Host(fake_hip.compile_host(str(tmp_path_factory.mktemp("host"))))


@pytest.mark.parametrize("n", [1, 300, 512, 513, 1024, 2048, 2049, 20_000])
def test_the_lanes_timed_are_the_lanes_launched(host, n):
    """The library's own choice for the configuration the tuner passes."""
    for lanes in (64, 128, 256, 512):
        host.reset()
        ctx = host.context(**tune._launch_config(dict(tune.DEFAULT, lanes=lanes), n, "exact"))
        g = host.graph(ctx)
        assert host.align(ctx, g, n=n) == 0 and host.launches()[0][1] == lanes
        host.lib.gwfa_graph_destroy(g)
        host.lib.gwfa_ctx_destroy(ctx)


def test_given_workgroups_and_pruned_modes_are_timed_as_configured():
    cfg = dict(tune.DEFAULT, groups=768)
    assert tune._launch_config(cfg, 100, "exact") is cfg
    assert tune._launch_config(tune.DEFAULT, 100, "heuristic") is tune.DEFAULT
