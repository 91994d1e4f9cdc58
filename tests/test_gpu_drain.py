"""Draining the lattice arcs of many channels in one call: around the numbers of channels at which the
kernel and its grid change, into a buffer that is too small, and after a drain has moved the rings on."""
import numpy as np
import pytest

import synth
from test_gpu_parity import B, torch_cuda  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 16, 17, 63, 64, 65, 130])
def test_batch_drains_what_single_drains_do(torch_cuda, B, n):  # noqa: F811
    torch = torch_cuda
    cfg = synth.configs()[0]
    graph = B.WfstGraph(synth.make_graph(cfg.graph))
    rng = np.random.default_rng(n)
    decs = [B.WfstDecoder(graph, 8.0, 4.0, 2000, num_channels=n, max_lanes=n, max_frames=20, token_capacity=4096,
                          history_capacity=40_000, lattice_capacity=12_000, lattice_on=True) for _ in range(2)]
    channels = rng.permutation(n).astype(np.int32)
    for d in decs:
        d.init_channels(channels)
    for chunk in range(2):
        rows = [torch.from_numpy(rng.normal(-2.0, 1.0, (int(rng.integers(1, 7)), cfg.graph.num_pdfs)).astype(np.float32)).cuda() for _ in range(n)]
        for d in decs:
            d.advance(channels, rows)
        with pytest.raises(B.WfstError):
            decs[0].lattice_arcs_batch(channels, out_device=torch.empty((0, 3), dtype=torch.int32, device="cuda"))
        records, offsets = decs[0].lattice_arcs_batch(channels)
        assert offsets[-1] > 0
        for i, c in enumerate(channels):
            assert sorted(records[offsets[i]:offsets[i + 1]].tolist()) == sorted(decs[1].lattice_arcs(int(c)).tolist())
        again, offsets = decs[0].lattice_arcs_batch(channels)
        assert len(again) == 0 and not offsets.any()
