"""What a call waits for: the calls that promise to, until the decoder's earlier work is over; the
readouts of snapshots, until the snapshot is sealed and no longer."""
import numpy as np
import pytest

import oracle
import synth
from gpu_compare import compare_channel
from test_gpu_parity import B, torch_cuda  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def test_initialising_channels_waits_for_the_decoding(torch_cuda, B):  # noqa: F811
    """The call returns when the last advance call (about 20 ms on a stream of its own) is over: the
    caller may overwrite the scores at once."""
    torch = torch_cuda
    c = synth.configs()[0]
    g = synth.make_graph(c.graph)
    T = 1500
    rows = [c.loglikes(s, 0, T) for s in range(3)]
    dec = B.WfstDecoder(B.WfstGraph(g), c.beam, c.lattice_beam, c.max_active, num_channels=3, max_lanes=2, max_frames=T,
                        lattice_capacity=4_000_000)
    dec.init_channels([0, 1])
    dev = [torch.from_numpy(r).cuda() for r in rows]
    torch.cuda.synchronize()
    stream, other, over = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Event()
    with torch.cuda.stream(stream):
        dec.advance([0, 1], dev[:2])
        over.record()
    dec.init_channels([2])
    assert over.query(), "init_channels returned while an advance call was running"
    for t in dev[:2]:
        t.zero_()
    with torch.cuda.stream(other):                 # the new channel's frames follow on another stream
        dec.advance([2], [dev[2]])
    torch.cuda.synchronize()
    og = oracle.OracleGraph(g)
    for ch, r in enumerate(rows):
        od = oracle.OracleDecoder(og, c.beam, c.lattice_beam, c.max_active)
        od.advance(r)
        compare_channel(dec, ch, od, frames=range(0, T + 1, 50), label=f"ch{ch}")
