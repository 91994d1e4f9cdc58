"""What the decoder is timed on: decoding jobs as a user's program runs them, through the Python binding.

A pass starts the streams of the job (wfst_decode_init_channels), feeds them their acoustic scores, and takes the results
the way the job's user takes them.  Four ways of feeding are covered:

  offline    whole utterances in one advance call, then the best paths and, with lattices on, the final lattices;
  online     one advance call over many chunks whose boundaries are read out beside the decoding (snapshots): the best path
             of every stream at every boundary and the boundary's lattice arcs, handed over in device memory;
  lockstep   one advance call per chunk, with the same readouts after each, from the live state;
  mux        more streams than lanes, taking turns chunk by chunk through the multiplexer, then the best paths.

Graphs, beams, limits and chunk lengths are those of synth.configs(): the 1000-state, the 200k-state and the 8M-state graph
(the 50M-state one is left out because building it takes longer than everything else here).  The graph is loaded once, as a
program does that decodes with one model; the seed decides the streams' scores and lengths.

Lattice arcs come in no particular order, so a pass puts the ones that it returns into (stream, frame, arc) order, on the
GPU; results whose number depends on the data stand at the front of buffers whose size does not.  Everything is compared bit for bit: costs are single fp32 additions in a fixed order, and minima do not depend on it."""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import synth
from paper_1910_10032_amd import binding as B

_CONFIGS = dict(zip(("tiny", "mid", "hclg"), synth.configs()[:3]))


def _case(name, mode, graph, streams, frames_lo, frames_hi, beam, max_active, lattice_beam=6.0, chunk=0, lattice=True,
          lanes=0, approximate=False, workgroups=0):
    c = dict(name=name, mode=mode, graph=graph, streams=streams, frames_lo=frames_lo, frames_hi=frames_hi, chunk=chunk,
             beam=beam, max_active=max_active, lattice=lattice, lattice_beam=lattice_beam, lanes=lanes or streams,
             approximate=approximate, workgroups=workgroups)
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # the smallest call: one stream, the first ten frames, and what has been recognised so far (a command word, a test)
        _case("tiny_first_chunk", "lockstep", "tiny", 1, 10, 10, 12.0, 2000, chunk=10, lattice=False),
        # a whole utterance on a small graph (grammar, command set), with its lattice
        _case("tiny_utterance", "offline", "tiny", 1, 300, 300, 12.0, 2000),
        # one utterance on a dense graph where max-active binds in every frame: rescoring or evaluating single files
        _case("mid_utterance", "offline", "mid", 1, 400, 400, 15.0, 7000, lattice_beam=8.0),
        # the same with several workgroups on the lane, the option for single heavy streams
        _case("mid_utterance_shared_lane", "offline", "mid", 1, 400, 400, 15.0, 7000, lattice_beam=8.0, workgroups=16),
        # one speaker dictating on the large graph: a partial result and its lattice arcs after every 0.3 s
        _case("hclg_dictation", "lockstep", "hclg", 1, 360, 360, 13.0, 7000, chunk=30),
        # an archive: a batch of whole utterances of all lengths, with lattices
        _case("hclg_offline_100", "offline", "hclg", 100, 500, 1500, 15.0, 10000, lattice_beam=8.0),
        # a full online service: 500 streams, partial results and lattice arcs at every 50-frame boundary
        _case("hclg_online_500", "online", "hclg", 500, 800, 800, 13.0, 7000, chunk=50),
        # the same service written the plain way: a call per chunk, read out before the next
        _case("hclg_lockstep_500", "lockstep", "hclg", 500, 100, 100, 13.0, 7000, chunk=50),
        # the most accurate setting: a wide beam, so that frames are large and max-active binds
        _case("hclg_wide_beam", "offline", "hclg", 150, 60, 140, 18.0, 7000),
        # one-best transcription at the highest rate: more streams than fit the chip at once, short beam, no lattices
        _case("hclg_one_best_1000", "offline", "hclg", 1000, 100, 300, 12.0, 7000, lattice=False),
        # the approximate cut where it is meant to help: a wide beam and a tight limit
        _case("hclg_approximate", "offline", "hclg", 64, 100, 200, 18.0, 2000, approximate=True),
        # three times as many callers as lanes, each sending quarter-second chunks
        _case("hclg_callers_on_lanes", "mux", "hclg", 300, 100, 100, 13.0, 7000, chunk=25, lattice=False, lanes=100),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    graph = rng.choice(("tiny", "mid", "hclg", "hclg", "hclg"))
    mode = rng.choice(("offline", "offline", "online", "lockstep", "mux"))
    most_streams = {"tiny": 64, "mid": 8, "hclg": 1000 if mode == "offline" else 500}[graph]
    streams = _log_uniform(rng, 1, most_streams)
    beam = round(rng.uniform(*{"tiny": (8.0, 12.0), "mid": (10.0, 15.0), "hclg": (10.0, 18.0)}[graph]), 2)
    max_active = {"tiny": 2000, "mid": 7000, "hclg": rng.choice((2000, 7000, 10000))}[graph]
    hi = _log_uniform(rng, 10, 1500)
    # no job longer than the longest listed one; streams beyond the number of compute units take turns
    us_per_frame = max(streams / 250, 1.0) * max(20.0, 0.025 * _arcs_per_frame(graph, beam))
    while hi > 10 and hi * us_per_frame > 60_000:
        hi = max(10, hi * 3 // 4)
    lo = hi if mode != "offline" else max(5, int(hi * rng.uniform(0.3, 1.0)))
    chunk = 0 if mode == "offline" else max(5, min(hi, rng.randint(10, 60)), -(-hi // 40))
    workgroups = rng.choice((0, 0, 7, 16)) if graph == "mid" and mode == "offline" else 0
    lanes = max(1, -(-streams // rng.choice((1, 2, 3)))) if mode == "mux" else streams
    return _case(None, mode, graph, streams, lo, hi, beam, max_active, lattice_beam=rng.choice((6.0, 8.0)), chunk=chunk,
                 lattice=mode != "mux" and rng.random() < 0.7, lanes=lanes, approximate=rng.random() < 0.15, workgroups=workgroups)


# ---- sizes -----------------------------------------------------------------------------------------------------------
# Mean number of arcs expanded per stream and frame, as the decoder counts them on these inputs, by beam.
_ARCS = {"tiny": ((8.0, 300.0), (12.0, 2273.0)), "mid": ((10.0, 3000.0), (15.0, 41885.0)),
         "hclg": ((10.0, 111.5), (12.0, 352.0), (13.0, 625.0), (15.0, 1777.0), (18.0, 7862.0))}


def _arcs_per_frame(graph, beam):
    pts = _ARCS[graph]
    return float(np.exp(np.interp(beam, [p[0] for p in pts], [math.log(p[1]) for p in pts])))


def work(case):
    """Per arc its 12-byte record and one score, per kept token its state's record and the token written and read again,
    12 bytes per lattice arc; three operations per arc."""
    frames = case["streams"] * (case["frames_lo"] + case["frames_hi"]) / 2
    arcs = _arcs_per_frame(case["graph"], case["beam"])
    tokens = min(0.35 * arcs, case["max_active"])
    lattice_arcs = 0.35 * arcs if case["lattice"] else 0.0
    return {"bytes": frames * (16 * arcs + 44 * tokens + 12 * lattice_arcs), "flops": frames * 3 * arcs}


def tolerance(case):
    return "exact"


def _capacities(case):
    """Buffer sizes with room for the busiest stream: tokens and lattice arcs of a frame, candidates before pruning."""
    graph, ma, frames = case["graph"], case["max_active"], case["frames_hi"]
    grow = math.exp(0.8 * (case["beam"] - 13.0))
    kept = ma + ma // 4 + 64 if case["approximate"] else ma
    if graph == "hclg":
        tokens, arcs = min(kept, max(800, int(800 * grow))), max(600, min(20000, int(600 * grow)))
        candidates = 16384 if case["beam"] <= 13 else 32768 if case["beam"] <= 15 else 65536
    else:
        tokens, arcs, candidates = kept, {"tiny": 4000, "mid": 30000}[graph], {"tiny": 4096, "mid": 65536}[graph]
    buffered = frames if case["mode"] == "offline" else case["chunk"]        # frames whose lattice arcs wait for a readout
    caps = dict(token_capacity=candidates, history_capacity=tokens * (frames + 1) + 4 * ma,
                lattice_capacity=arcs * buffered + 100_000)
    if case["mode"] == "online" and case["lattice"]:
        caps["snapshot_blocks"] = -(-frames // case["chunk"])
        caps["snapshot_block_capacity"] = max(caps["lattice_capacity"], case["streams"] * case["chunk"] * arcs // 2)
    return caps


# ---- one pass --------------------------------------------------------------------------------------------------------
_graphs = {}


def _graph(name):
    if name not in _graphs:
        _graphs[name] = B.WfstGraph(synth.make_graph(_CONFIGS[name].graph))
    return _graphs[name]


class _Job:
    """A decoder, its streams' scores on the GPU, and the arguments of the calls."""

    def __init__(self, case, seed):
        cfg = _CONFIGS[case["graph"]]
        rng = random.Random(seed)
        n, pdfs = case["streams"], cfg.graph.num_pdfs
        self.mode, self.chunk, self.lattice = case["mode"], case["chunk"], case["lattice"]
        self.lens = np.array([rng.randint(case["frames_lo"], case["frames_hi"]) for _ in range(n)], np.int32)
        first = np.concatenate([[0], np.cumsum(self.lens, dtype=np.int64)])
        self.scores = torch.empty((int(first[-1]), pdfs), dtype=torch.float32, device="cuda")
        score_seed = rng.getrandbits(48)
        for s in range(n):
            synth.device_loglikes(self.scores[first[s]:first[s + 1]], score_seed, s, 0, cfg.ll_mu, cfg.ll_sigma, cfg.ll_boost)
        self.caps = _capacities(case)
        self.decoder = B.WfstDecoder(_graph(case["graph"]), case["beam"], case["lattice_beam"], case["max_active"],
                                     num_channels=n, max_lanes=case["lanes"], max_frames=case["frames_hi"],
                                     lattice_on=case["lattice"], approximate=case["approximate"],
                                     lane_workgroups=case["workgroups"], **self.caps)
        self.channels = np.arange(n, dtype=np.int32)
        self.words_cap = case["frames_hi"] // 2 + 64
        self.final_cap = int(n * case["frames_hi"] * {"tiny": 100, "mid": 50, "hclg": 8}[case["graph"]]) + 1000
        self.rows = self.scores.data_ptr() + first[:-1].astype(np.uint64) * np.uint64(4 * pdfs)
        self.strides = np.full(n, pdfs, np.int32)
        streams = [self.scores[first[s]:first[s + 1]] for s in range(n)]
        self.chunks = []                                  # per call: the tensors of scores that the acoustic model delivered
        if self.mode == "offline":
            self.chunks = [streams]
        elif self.mode == "lockstep":
            self.chunks = [[t[f:f + self.chunk] for t in streams] for f in range(0, int(self.lens.max()), self.chunk)]
        self.arcs = None                                  # where lattice arcs are delivered, in device memory
        if self.lattice and self.mode != "offline":
            room = self.caps["snapshot_block_capacity"] if self.mode == "online" else n * self.caps["lattice_capacity"] // 2 + 100_000
            self.arcs = torch.empty((room, 3), dtype=torch.int32, device="cuda")
        self.mux = B.WfstMux(self.decoder) if self.mode == "mux" else None


def prepare(case, seed):
    return _Job(case, seed)


def _in_order(records, owner, room):
    """Lattice arcs ({frame, arc, extra cost} rows) of the streams `owner`, sorted by (stream, frame, arc), in buffers of `room`."""
    keys = torch.full((room,), -1, dtype=torch.int64, device="cuda")
    extra = torch.zeros(room, dtype=torch.float32, device="cuda")
    key, at = torch.sort((owner << 43) | (records[:, 0].long() << 31) | records[:, 1].long())
    keys[:len(key)] = key
    extra[:len(key)] = records[:, 2].view(torch.float32)[at]
    return keys, extra


def _owner(counts, streams=None):
    """The stream of each record, for runs of `counts` records one behind the other."""
    counts = torch.from_numpy(np.ascontiguousarray(counts)).cuda()
    streams = torch.arange(len(counts), device="cuda") if streams is None else torch.from_numpy(streams).cuda()
    return torch.repeat_interleave(streams, counts)


class _Paths:
    """Best paths as they come, readout by readout."""

    def __init__(self):
        self.words, self.rest = [], []

    def add(self, got):
        words, n_words, *rest = got
        words[np.arange(words.shape[1]) >= n_words[:, None]] = 0
        self.words.append(words)
        self.rest.append((n_words, *rest))

    def all(self):
        names = ("n_words", "total_cost", "reached_final", "status")
        return dict(zip(names, (np.stack(v) for v in zip(*self.rest))), words=np.stack(self.words))


def run(job):
    dec, ch, paths = job.decoder, job.channels, _Paths()
    dec.init_channels(ch)
    out = {}
    if job.mode == "offline":
        dec.advance(ch, job.chunks[0])
        paths.add(dec.best_path_batch(ch, use_final=True, words_cap=job.words_cap, raw=True))
        if job.lattice:
            records, offsets, infos, status = dec.final_lattice_batch(ch, use_final=True)
            flat = torch.from_numpy(records.view(np.int32).reshape(-1, 3)).cuda()
            out["lattice"] = _in_order(flat, _owner(np.diff(offsets)), job.final_cap)
            out["lattice_info"] = [offsets, status, np.array([i["best_cost"] for i in infos], np.float32),
                                   np.array([i["arcs_in"] for i in infos], np.int64)]
    elif job.mode == "online":
        stream = torch.cuda.current_stream().cuda_stream
        first, count = dec.advance_ptrs(ch, job.rows, job.strides, job.lens, stream, snapshot_every=job.chunk)
        counts = []
        for k in range(first, first + count):
            paths.add(dec.best_path_batch(ch, use_final=False, words_cap=job.words_cap, raw=True, snapshot=k))
            if job.lattice:
                got = dec.snapshot_lattice_arcs(k, ch, out_device=job.arcs, copy=k == first + count - 1)
                counts.append(got["counts"])
        if job.lattice:
            by_place = np.argsort(got["starts"] * 2 + (got["counts"] > 0), kind="stable")     # (empty runs may share a start)
            out["lattice"] = _in_order(job.arcs[:got["total"]], _owner(got["counts"][by_place], by_place), len(job.arcs))
            out["lattice_counts"] = np.stack(counts)
    elif job.mode == "lockstep":
        offsets = []
        for scores in job.chunks:
            dec.advance(ch, scores)
            paths.add(dec.best_path_batch(ch, use_final=False, words_cap=job.words_cap, raw=True))
            if job.lattice:
                offsets.append(dec.lattice_arcs_batch(ch, out_device=job.arcs))
        if job.lattice:
            out["lattice"] = _in_order(job.arcs[:offsets[-1][-1]], _owner(np.diff(offsets[-1])), len(job.arcs))
            out["lattice_offsets"] = np.stack(offsets)
    else:
        stream = torch.cuda.current_stream().cuda_stream
        pitch, rows, lens = int(job.strides[0]), job.rows.tolist(), job.lens.tolist()
        for f in range(0, max(lens), job.chunk):
            for c, (row, length) in enumerate(zip(rows, lens)):
                if f < length:
                    job.mux.submit(c, row + 4 * pitch * f, pitch, min(job.chunk, length - f))
            while job.mux.pending():
                job.mux.step(stream)
        paths.add(dec.best_path_batch(ch, use_final=True, words_cap=job.words_cap, raw=True))
    return dict(out, **paths.all())
