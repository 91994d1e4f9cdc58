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


@pytest.mark.parametrize("words_cap", [464, 4096])
def test_the_first_readout_of_a_new_decoder_runs_beside_the_decoding(torch_cuda, B, words_cap):  # noqa: F811
    """The first snapshots of an advance call of about 20 ms are sealed after less than 1 ms.  Reading
    them grows the decoder's buffers (twice), which must not wait for the call; one later readout with
    the buffers of both sizes, and all of them against the oracle."""
    torch = torch_cuda
    c = synth.configs()[0]
    g = synth.make_graph(c.graph)
    n, T, chunk = 64, 1500, 30
    rows = [c.loglikes(s, 0, T) for s in range(n)]
    dec = B.WfstDecoder(B.WfstGraph(g), c.beam, c.lattice_beam, c.max_active, num_channels=n, max_lanes=n, max_frames=T,
                        lattice_on=False)
    chans = list(range(n))
    dec.init_channels(chans)
    dev = [torch.from_numpy(r).cuda() for r in rows]
    torch.cuda.synchronize()
    over, got = torch.cuda.Event(), []
    with torch.cuda.stream(torch.cuda.Stream()):
        first, _ = dec.advance(chans, dev, snapshot_every=chunk)
        over.record()
    for k, cap in ((0, words_cap), (1, 2 * words_cap)):
        got.append((k, dec.best_path_batch(chans, use_final=False, words_cap=cap, snapshot=first + k)))
        assert not over.query(), f"the readout of snapshot {k} waited for the advance call"
    got.append((49, dec.best_path_batch(chans, use_final=False, words_cap=words_cap, snapshot=first + 49)))
    og = oracle.OracleGraph(g)
    for ch in (0, 1, 31, 63):
        od = oracle.OracleDecoder(og, c.beam, c.lattice_beam, c.max_active)
        done = 0
        for k, res in got:
            od.advance(rows[ch][done:(k + 1) * chunk])
            done = (k + 1) * chunk
            want = od.best_path(False)
            assert res[ch]["status"] == 0 and np.array_equal(res[ch]["words"], want["words"]), f"snapshot {k} ch {ch}"
            assert np.float32(res[ch]["total_cost"]).view(np.uint32) == np.float32(want["total_cost"]).view(np.uint32)
