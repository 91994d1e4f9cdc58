"""States whose places in the state table are the same: more of them than are looked at before a frame is given up."""
import numpy as np
import pytest

from gpu_compare import compare_channel
from helpers import G
from test_gpu_parity import B, F32, run_pair, torch_cuda  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def one_slot(K, seed):
    """K states with the same first slot in a table of 2048 (two neighbouring ones in 4096).  State 0 leads to all of them;
    each leads to one of them, and to the next one without a score."""
    rng = np.random.default_rng(seed)
    home, chosen, handle = None, [], 1 + K                 # (the handle of state 1: state 0's header and arcs lie before it)
    s = 1
    while len(chosen) < K:
        h = (handle * 2654435761 & 0xFFFFFFFF) >> 21
        home = h if home is None else home
        if h == home:
            chosen.append(s)
        handle += 3 if h == home and len(chosen) < K else 2
        s += 1
    N, chosen = s, np.array(chosen)
    degree = np.ones(N, np.int64)
    degree[0] = K
    degree[chosen[:-1]] = 2
    off = np.concatenate([[0], np.cumsum(degree)])
    E = int(off[-1])
    ilabel, olabel = rng.integers(1, 4, E).astype(np.int32), rng.integers(0, 5, E).astype(np.int32)
    weight, nextstate = rng.integers(0, 4, E).astype(np.float32), rng.choice(chosen, E).astype(np.int32)
    nextstate[:K] = chosen
    eps = off[chosen[:-1]] + 1
    ilabel[eps], weight[eps], nextstate[eps] = 0, 1.0, chosen[1:]
    final = np.full(N, np.inf, np.float32)
    final[chosen[::3]] = 0.0
    return G(N, E, 0, 3, off.astype(np.int64), ilabel, olabel, weight, nextstate, final), [-rng.integers(0, 2, size=(4, 3)).astype(F32)]


@pytest.mark.parametrize("threads,workgroups", [(256, 1), (512, 1), (1024, 1), (0, 3)])
@pytest.mark.parametrize("K,alpha", [(40, 20000), (300, 20000), (300, 100)])
def test_states_with_the_same_first_slot(torch_cuda, B, K, alpha, threads, workgroups):  # noqa: F811
    g, rows = one_slot(K, seed=K)
    dec, ods, _ = run_pair(torch_cuda, B, g, rows, beam=30.0, lbeam=2.0, alpha=alpha, token_capacity=1 << 13,
                           lattice_capacity=1 << 16, lane_threads=threads, lane_workgroups=workgroups)
    compare_channel(dec, 0, ods[0], label=f"{K} states, alpha {alpha}, {threads} threads, {workgroups} workgroups")
