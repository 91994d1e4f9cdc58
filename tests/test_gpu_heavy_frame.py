"""The frame with thousands of tokens, worked through by one workgroup or a team of them: at the sizes
where a table fills up, with chains of epsilon arcs between states of different owners, ties at the
max-active cut, degrees and pdf ids that do not fit the arc records, and tight buffers."""
import numpy as np
import pytest

import oracle
import synth
from gpu_compare import compare_channel
from test_gpu_parity import (B, F32, _check_paths, _check_snapshot_lattice, _oracle_lattice_of_frames, run_pair,  # noqa: F401
                             torch_cuda)  # (fixtures)

pytestmark = pytest.mark.gpu


def layers(K, seed, wmax=6, chain=5, num_pdfs=7, wide=(), many_eps=()):
    """A start state that fans out to K states, which reach each other at random and are linked by
    epsilon chains; `wide`: states with thousands of emitting arcs; `many_eps`: with dozens of epsilon arcs."""
    from helpers import graph_from_arcs
    rng = np.random.default_rng(seed)
    hubs = -(-K // 3000)                                   # the fan goes over a few hubs in the first frame
    first = 1 + hubs
    arcs = [(0, 1 + i, 1, 0, 0.0) for i in range(hubs)]
    arcs += [(1 + i % hubs, first + i, 1 + int(rng.integers(0, num_pdfs)), 1 + i % 5, float(rng.integers(0, wmax))) for i in range(K)]
    dst, pdf, w = rng.integers(0, K, size=(K, 2)), rng.integers(0, num_pdfs, size=(K, 2)), rng.integers(0, wmax, size=(K, 2))
    for i in range(K):
        arcs += [(first + i, first + int(dst[i, k]), 1 + int(pdf[i, k]), 0, float(w[i, k])) for k in range(2)]
        if i % chain and i + 1 < K:
            arcs.append((first + i, first + i + 1, 0, 3, 0.25))
    for s in wide:
        arcs += [(first + s, first + int(d), 1 + int(d) % num_pdfs, 0, float(int(d) % wmax)) for d in rng.integers(0, K, size=4200)]
    for s in many_eps:
        arcs += [(first + s, first + s + 1 + int(d), 0, 0, 0.5) for d in rng.integers(0, K - s - 1, size=40)]
    g = graph_from_arcs(first + K, arcs, num_pdfs=num_pdfs, finals={first + K - 1: 0.0, first: 1.0})
    return g, [-rng.integers(0, 3, size=(5, num_pdfs)).astype(F32)]


@pytest.mark.parametrize("kw,sizes", [(dict(lane_threads=256), (1536, 1537, 3071, 3072, 3073)),
                                      (dict(lane_threads=512), (1536, 1537, 3071, 3072, 3073)),
                                      (dict(lane_threads=1024, lane_workgroups=1), (3072, 3073, 6143, 6144, 6145)),
                                      (dict(lane_workgroups=2), (6145, 11000, 13000)),
                                      (dict(lane_workgroups=7), (3073, 9000, 30000)),
                                      (dict(), (3073, 20000))])
def test_frames_around_the_size_of_the_tables(torch_cuda, B, kw, sizes):  # noqa: F811
    for K in sizes:
        g, rows = layers(K, seed=K)
        dec, ods, _ = run_pair(torch_cuda, B, g, rows, beam=40.0, lbeam=3.0, alpha=40000, token_capacity=1 << 17,
                               lattice_capacity=1 << 20, **kw)
        assert ods[0].max_tokens >= K
        compare_channel(dec, 0, ods[0], label=f"K={K} {kw}")


@pytest.mark.parametrize("kw", [dict(lane_threads=256), dict(lane_threads=512), dict(lane_workgroups=1), dict(lane_workgroups=3), dict(lane_workgroups=16)])
@pytest.mark.parametrize("alpha", [1, 500, 800, 1200, 2500])
def test_ties_at_the_cut(torch_cuda, B, kw, alpha):  # noqa: F811
    """Integer costs of two values: thousands of equal costs at the cut, decided by the state id.  The
    selection ends with a list of the pairs left at the cut: with 2900 states and a limit of 500 to
    1200 it is 288 to 494 pairs long in nearly every frame, more than 256 threads and at most HEAVY_LIST."""
    g, rows = layers(2900 if "lane_threads" in kw else 5000, seed=alpha, wmax=2)
    dec, ods, _ = run_pair(torch_cuda, B, g, [np.round(r / 4) for r in rows], beam=40.0, lbeam=3.0, alpha=alpha, token_capacity=1 << 15,
                           lattice_capacity=1 << 20, **kw)
    compare_channel(dec, 0, ods[0], label=f"alpha={alpha} {kw}")


@pytest.mark.parametrize("kw", [dict(lane_threads=256), dict(lane_threads=512), dict(lane_workgroups=1), dict(lane_workgroups=5)])
@pytest.mark.parametrize("num_pdfs", [7, 70000])
def test_degrees_and_pdf_ids_that_do_not_fit_the_records(torch_cuda, B, kw, num_pdfs):  # noqa: F811
    g, rows = layers(2500, seed=3, num_pdfs=num_pdfs, wide=(5, 77), many_eps=(0, 9, 1000))
    dec, ods, _ = run_pair(torch_cuda, B, g, rows, beam=30.0, lbeam=3.0, alpha=20000, token_capacity=1 << 15, lattice_capacity=1 << 20, **kw)
    compare_channel(dec, 0, ods[0], label=f"pdfs={num_pdfs} {kw}")


@pytest.mark.parametrize("kw", [dict(lane_workgroups=1), dict(lane_workgroups=16)])
@pytest.mark.parametrize("token_capacity", [4200, 6000, 9000])
def test_tight_buffers_and_chunked_calls(torch_cuda, B, kw, token_capacity):  # noqa: F811
    """Buckets and lists that overflow: the frame is redone in the general form; several streams, in chunks."""
    cases = [layers(4000, seed=s) for s in range(3)]
    rows = [c[1][0][:n] for c, n in zip(cases, (5, 3, 4))]
    dec, ods, _ = run_pair(torch_cuda, B, cases[0][0], rows, beam=40.0, lbeam=3.0, alpha=3000, token_capacity=token_capacity, aux_capacity=20000,
                           lattice_capacity=1 << 18, chunks=[2, 2, 1], **kw)
    for ch, od in enumerate(ods):
        compare_channel(dec, ch, od, label=f"capacity={token_capacity} {kw} ch{ch}")


def test_the_approximate_cut_is_the_same_in_every_form(torch_cuda, B):  # noqa: F811
    g, rows = layers(2900, seed=8)
    got = []
    for kw in (dict(frame_form=1), dict(lane_threads=512), dict(lane_workgroups=1), dict(lane_workgroups=4)):
        dec = run_pair(torch_cuda, B, g, rows, beam=40.0, lbeam=3.0, alpha=1000, approximate=True, token_capacity=1 << 15,
                       lattice_capacity=1 << 20, **kw)[0]
        got.append([np.sort(dec.tokens(0, f), order="state") for f in range(6)] + [np.sort(dec.lattice_arcs(0), order=("frame", "arc"))])
    for other in got[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(got[0], other))


@pytest.mark.parametrize("kw", [dict(lane_threads=512), dict(), dict(lane_workgroups=2), dict(lane_workgroups=16)])
def test_snapshots_between_heavy_frames(torch_cuda, B, kw):  # noqa: F811
    """Lanes seal a snapshot after every 7 frames of thousands of tokens (most of them written by the
    other workgroups of the lane's team): the best paths and lattice arcs of each, read beside the
    decoding, and the whole history afterwards."""
    torch = torch_cuda
    c = synth.configs()[1]
    g = synth.make_graph(c.graph)
    lens, chunk = [42, 30], 7
    rows = [c.loglikes(s, 0, n) for s, n in enumerate(lens)]
    og = oracle.OracleGraph(g)
    step = [oracle.OracleDecoder(og, c.beam, c.lattice_beam, c.max_active) for _ in lens]
    dec = B.WfstDecoder(B.WfstGraph(g), c.beam, c.lattice_beam, c.max_active, num_channels=2, max_lanes=2, max_frames=42,
                        token_capacity=1 << 16, lattice_capacity=1 << 20, snapshot_blocks=6, snapshot_block_capacity=1 << 20, **kw)
    dec.init_channels([0, 1])
    dev = [torch.from_numpy(r).cuda() for r in rows]
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        first, count = dec.advance([0, 1], dev, snapshot_every=chunk)
    assert count == 6
    for j in range(count):
        for od, r in zip(step, rows):
            if len(r) > j * chunk:
                od.advance(r[j * chunk:(j + 1) * chunk])
        _check_paths(dec.best_path_batch([0, 1], use_final=False, snapshot=first + j), step, False, f"snapshot {j} {kw}")
        lo = lambda ch: min(0 if j == 0 else j * chunk + 1, lens[ch] + 1)
        hi = lambda ch: min((j + 1) * chunk, lens[ch]) + 1
        r, covered = _check_snapshot_lattice(dec, first + j, [0, 1], lambda ch: _oracle_lattice_of_frames(step[ch], lo(ch), hi(ch)),
                                             f"snapshot {j} {kw}")
        assert covered == r["total"]
    torch.cuda.synchronize()
    for ch, od in enumerate(step):
        assert od.max_tokens_pre_prune > c.max_active
        compare_channel(dec, ch, od, label=f"ch{ch} {kw}", lattice=False)
