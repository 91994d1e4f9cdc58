"""The LDS-resident frame at the sizes where its structures fill up: emitting arcs of a frame (one
tile, two tiles, too many), epsilon arcs listed, states without an emitting arc among the tokens."""
import numpy as np
import pytest

from gpu_compare import compare_channel
from test_gpu_parity import B, F32, run_pair, torch_cuda  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def fan(n_arcs, n_eps, seed):
    """States reached in frame 1 whose arcs take exactly n_arcs positions in frame 2 (three each, every
    ninth state has none and takes one), n_eps epsilon arcs among them, two per state where possible."""
    from helpers import graph_from_arcs
    rng = np.random.default_rng(seed)
    degree = []
    while sum(max(d, 1) for d in degree) < n_arcs:
        degree.append(0 if len(degree) % 9 == 4 else 3)
    degree[-1] = max(1, degree[-1] - (sum(max(d, 1) for d in degree) - n_arcs))
    K = len(degree)
    end = K + 1
    arcs = [(0, 1 + i, 1 + i % 3, 1 + i % 5, float(rng.integers(0, 4))) for i in range(K)]
    for i, d in enumerate(degree):
        arcs += [(1 + i, (1 + int(rng.integers(0, K))) if k else 1 + i, 1 + int(rng.integers(0, 3)), 0, float(rng.integers(1, 4)))
                 for k in range(d)]
    left = n_eps
    for i in range(K):
        for _ in range(min(2, left)):
            arcs.append((1 + i, end, 0, 2, 0.5))
            left -= 1
    arcs.append((end, end, 1, 0, 0.25))
    g = graph_from_arcs(K + 2, arcs, num_pdfs=3, finals={end: 0.0, 1: 1.0})
    return g, [-rng.integers(0, 2, size=(4, 3)).astype(F32)]


CASES = [(t, n, 16) for t in (256, 512, 1024) for n in (t - 1, t, t + 1, 2 * t, 2 * t + 1, 4 * t - 1, 4 * t, 4 * t + 1, 8 * t - 1, 8 * t, 8 * t + 1)]
CASES += [(t, 4 * t if t < 1024 else 6000, e) for t in (256, 512, 1024) for e in ((1279, 1280, 1281) if t < 1024 else (2559, 2560, 2561))]


@pytest.mark.parametrize("threads,n_arcs,n_eps", CASES)
def test_frames_at_the_limits_of_the_arc_and_epsilon_lists(torch_cuda, B, threads, n_arcs, n_eps):  # noqa: F811
    g, rows = fan(n_arcs, n_eps, seed=n_arcs + n_eps)
    dec, ods, _ = run_pair(torch_cuda, B, g, rows, beam=30.0, lbeam=2.0, alpha=20000, token_capacity=1 << 14,
                           lattice_capacity=1 << 18, lane_threads=threads)
    compare_channel(dec, 0, ods[0], label=f"arcs={n_arcs} eps={n_eps} threads={threads}")


@pytest.mark.parametrize("alpha", [1, 100, 700])
@pytest.mark.parametrize("threads", [256, 512, 1024])
def test_max_active_cut_renumbers_the_tokens(torch_cuda, B, threads, alpha):  # noqa: F811
    g, rows = fan(2 * threads + 37, 100, seed=alpha)
    dec, ods, _ = run_pair(torch_cuda, B, g, rows, beam=30.0, lbeam=2.0, alpha=alpha, token_capacity=1 << 14,
                           lattice_capacity=1 << 18, lane_threads=threads)
    compare_channel(dec, 0, ods[0], label=f"alpha={alpha} threads={threads}")
