"""GPU: which pruned queries are run again off the small arenas, and what comes
of them: those that outgrow the lists there, and those too long for the
directory there, which go to the configured arenas at once.

Bar: results as in the narrow wavefronts' tests, bit for bit against the
oracle; exact counts of queries run again."""
import numpy as np
import pytest

from tests.test_gpu_narrow import G, _compare, _dna  # noqa: F401 (G: fixture)

pytestmark = pytest.mark.gpu


def wide_hub_case(rng, deg):
    """A vertex with `deg` out-edges (a list of that many entries at score 0),
    a join, 900 bases without errors (every other diagonal then lags by more
    than 1,025), errors at the end."""
    labels = [_dna(rng, 60)] + [_dna(rng, int(rng.integers(20, 40))) for _ in range(deg)] + [_dna(rng, 1000)]
    edges = [(0, 1 + j) for j in range(deg)] + [(1 + j, deg + 1) for j in range(deg)]
    q = list(labels[0] + labels[1 + int(rng.integers(0, deg))] + labels[-1])
    for p in (30, 12, 5):
        q[-p] = "ACGT"[("ACGT".index(q[-p]) + 1) % 4]
    return labels, edges, "".join(q).encode(), 0


@pytest.mark.parametrize("a_diff,again", [(40, 3), (1024, 3), (1025, 0)])
def test_lists_that_outgrow_the_small_arenas(G, a_diff, again):  # noqa: F811
    """5,000 entries: more than the small arenas' 4,096, fewer than the
    configured 32,768, where a lag of 1,025 starts."""
    gw, ctx = G
    ctx.config(lanes=64)
    rng = np.random.default_rng(8700)
    cases = [wide_hub_case(rng, d) for d in (5000, 40, 5000, 1000, 5000, 1)]
    ctx.stats(reset=True)
    print(f"[gpu-first-tier] hubs, a_diff={a_diff}", flush=True)
    _compare(gw, ctx, cases, a_diff)
    assert ctx.stats()["reruns"] == again


@pytest.mark.parametrize("a_diff,again", [(50, 1), (263, 2), (400, 130), (1024, 130), (1025, 0)])
def test_queries_too_long_for_the_small_arenas(G, a_diff, again):  # noqa: F811
    """A graph of single bases (1.36, 2.05, 2.49 and 4.50 pages a base by the
    rule): half the directory, 8,192 pages, is for 6,018, 4,000, 3,290 and 1,819
    bases.  One or two of 130 queries are left to the configured arenas alone,
    from three on (more than 1 in 64) the others with them."""
    gw, ctx = G
    ctx.config(lanes=64)
    rng = np.random.default_rng(8800)
    cases = []
    for n in [300] * 126 + [1950, 3400, 5000, 6100]:
        labels = list(_dna(rng, n + 40))
        edges = [(i, i + 1) for i in range(n + 39)] + [(i, i + 2) for i in range(0, n, 97)]
        q = list("".join(labels[:n]))
        for p in rng.integers(0, n, size=12):
            q[p] = _dna(rng, 1)
        cases.append((labels, edges, "".join(q).encode(), 0))
    ctx.stats(reset=True)
    print(f"[gpu-first-tier] single-base graph, a_diff={a_diff}", flush=True)
    _compare(gw, ctx, cases, a_diff)
    assert ctx.stats()["reruns"] == again


@pytest.mark.parametrize("too_long,again", [(6, 6), (20, 600)])
def test_large_batches_are_judged_by_a_sample(G, too_long, again):  # noqa: F811
    """600 queries, longest first: of 256 places spread over them, 3 or 9 hold a
    query too long (4 are 1 in 64)."""
    gw, ctx = G
    ctx.config(lanes=64)
    rng = np.random.default_rng(8900)
    cases = []
    for n in [60] * (600 - too_long) + [1900] * too_long:
        labels = list(_dna(rng, n + 5))
        q = list("".join(labels[:n]))
        q[n // 2] = _dna(rng, 1)
        cases.append((labels, [(i, i + 1) for i in range(n + 4)], "".join(q).encode(), 0))
    ctx.stats(reset=True)
    print(f"[gpu-first-tier] 600 queries, {too_long} too long", flush=True)
    _compare(gw, ctx, cases, 1024)
    assert ctx.stats()["reruns"] == again
