"""HIP decode (tbs_decode) against the CPU oracle, element by element.

Every case runs under both frame-loop schedules: "frame" (a joiner GEMM kernel and a
search kernel per frame) and "stream" (persistent workgroups: one per stream, or for
the trivial graph with an fp32 joiner several per stream where the shape allows;
"stream1" forces one).  A shape
the per-stream kernel cannot hold must be refused with TBS_EUNSUPPORTED; such a run is
reported and skipped.

Parity rule (see parity.py): survivor traces identical up to the first frame with a
decision margin below MARGIN, and over whole streams where no decision is that close;
tokens, arcs and status identical on such streams; scores within 1e-4 (fp32 joiner) or
2e-2 (bf16 joiner, against the bf16-operand oracle).  Then every frame of every checked
stream is replayed: the oracle decides it again from the HIP path's own survivors of the
previous frame, and the HIP survivors must equal the oracle's bit for bit wherever that
frame's margin exceeds MARGIN (a valid selection elsewhere).  Each case asserts a floor
on the frames compared bit for bit.  MARGIN (1e-4 for fp32) is tighter
than the 1e-3 the tolerance allows: the fp32 path's per-decision score error is ~1e-6.
For the bf16 joiner, h rounds to bf16 from an fp32 tanh on the GPU and from an fp64 tanh
in the oracle; isolated elements then round to neighbouring bf16 values (logit error
~1e-4..1e-3), so its margin is 2e-3.
"""
import math

import numpy as np
import pytest

import oracle
from gpu_util import gpu_decode, say
from parity import check_trace_invariants, compare, replay_check
from paper_2211_00484_amd import synth

pytestmark = pytest.mark.gpu

FP32 = dict(margin=1e-4, score_tol=1e-4)
BF16 = dict(margin=2e-3, score_tol=2e-2)


SCHEDULES = ["frame", "stream"]


def _run(name_or_parts, beam, Ns, Nc, dtype="fp32", streams=None, nthreads=0, seed=0, B=None,
         schedule="frame", exact_floor=None):
    """Decodes on the GPU, compares with the oracle and replays every frame.  Returns
    (gpu, oracle, report).  exact_floor: the smallest fraction of the
    checked frames the replay must compare bit for bit (default: half of what the
    oracle's own margins predict)."""
    from paper_2211_00484_amd import tbs
    if isinstance(name_or_parts, str):
        w, inputs, model, graph = synth.make_workload(name_or_parts, seed=seed, B=B)
    else:
        inputs, model, graph = name_or_parts
    say(f"decode B={inputs.B} T={inputs.T} V={model.vocab_size} C={model.dim} "
        f"S={graph.num_states} beam={beam} Ns={Ns} Nc={Nc} {dtype} {schedule}")
    try:
        g = gpu_decode(model, graph, inputs, beam, Ns, Nc, dtype=dtype, schedule=schedule)
    except tbs.TbsError as e:
        if schedule == "stream" and e.status == -5:
            say(f"  not supported by the per-stream kernel: {e}")
            return None, None, None
        raise
    streams = list(range(inputs.B)) if streams is None else list(streams)
    o = oracle.decode(model, graph, inputs.encoder_out, inputs.lengths, beam, Ns, Nc,
                      bf16=(dtype == "bf16"), nthreads=nthreads, streams=streams)
    tol = BF16 if dtype == "bf16" else FP32
    rep = compare(g, o, model, graph, inputs.encoder_out, inputs.lengths, streams,
                  bf16=(dtype == "bf16"), **tol)
    check_trace_invariants(g["trace"], inputs.lengths, graph, model.vocab_size, Ns, min(Nc, Ns),
                           streams)
    say(f"  {rep}")
    rrep = replay_check(g, model, graph, inputs.encoder_out, inputs.lengths, streams, beam, Ns,
                        min(Nc, Ns), margin=tol["margin"], tol=tol["score_tol"],
                        bf16=(dtype == "bf16"), nthreads=nthreads)
    say(f"  {rrep}")
    predicted = sum(int((o.frame_margins[k, :inputs.lengths[b]] > tol["margin"]).sum())
                    for k, b in enumerate(streams))
    floor = (exact_floor * rrep.frames) if exact_floor is not None else 0.5 * predicted
    assert rrep.exact >= floor, f"only {rrep.exact} of {rrep.frames} frames compared bit for bit"
    return g, o, rep


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_tiny(dtype, schedule):
    _, _, rep = _run("tiny", math.inf, 4, 4, dtype, schedule=schedule)
    assert rep.streams == 2


@pytest.mark.parametrize("beam,Ns,Nc", [(math.inf, 1, 1), (1.0, 3, 2), (0.5, 8, 3), (2.0, 16, 16),
                                        (0.0, 4, 4), (math.inf, 12, 12)])
@pytest.mark.parametrize("schedule", SCHEDULES)
def test_tiny_params(beam, Ns, Nc, schedule):
    _run("tiny", beam, Ns, Nc, seed=3, schedule=schedule)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_ragged_and_empty_lengths(schedule):
    rng = np.random.default_rng(9)
    model = synth.make_model(rng, 16, 32, 0.1)
    inputs = synth.make_inputs(rng, 7, 25, 32)
    inputs.lengths[:] = [0, 25, 1, 13, 0, 24, 7]
    for b in range(inputs.B):
        inputs.encoder_out[b, inputs.lengths[b]:] = 0.0
    g, o, _ = _run((inputs, model, synth.trivial_graph(16)), math.inf, 4, 4, schedule=schedule)
    for b in (0, 4):
        assert g["ntok"][b] == 0 and g["scores"][b] == 0.0 and (g["tokens"][b] == -1).all()


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("seed", range(12))
def test_random_small_graphs(seed, schedule):
    rng = np.random.default_rng(100 + seed)
    V = int(rng.integers(3, 40))
    C = int(rng.integers(1, 70))
    S = int(rng.integers(1, 60))
    model = synth.make_model(rng, V, C, 0.4)
    inputs = synth.make_inputs(rng, 5, 40, C, length_range=(0, 40))
    graph = synth.random_small_graph(rng, S, V, max_degree=int(rng.integers(1, 12)),
                                     with_final=bool(seed % 2))
    beam = [math.inf, 3.0, 1.0][seed % 3]
    Ns = int(rng.integers(1, 33))
    Nc = int(rng.integers(1, Ns + 1))
    _run((inputs, model, graph), beam, Ns, Nc, dtype=["fp32", "bf16"][seed % 4 == 3],
         schedule=schedule)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_many_candidate_chunks(schedule):
    # 8 tuples x 2999 arcs: the per-stream candidate set spans many LDS merge passes.
    rng = np.random.default_rng(5)
    V, C = 3000, 48
    model = synth.make_model(rng, V, C, 0.2)
    inputs = synth.make_inputs(rng, 3, 12, C)
    _run((inputs, model, synth.trivial_graph(V)), math.inf, 8, 8, schedule=schedule)
    _run((inputs, model, synth.trivial_graph(V)), 2.0, 8, 3, schedule=schedule)
    # general graph over the same vocabulary: logits are gathered per arc
    graph = synth.random_small_graph(rng, 20, V, max_degree=400)
    _run((inputs, model, graph), 3.0, 16, 8, schedule=schedule)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_maximum_vocabulary(schedule):
    # V = 46,340, the largest vocabulary whose contexts a * V + b fit int32: the trivial
    # graph (725 vocabulary tiles per row) and a small graph whose labels reach V - 1
    rng = np.random.default_rng(21)
    V, C = 46340, 16
    model = synth.make_model(rng, V, C, 0.5)
    inputs = synth.make_inputs(rng, 2, 4, C)
    _run((inputs, model, synth.trivial_graph(V)), math.inf, 4, 4, schedule=schedule)
    graph = synth.random_small_graph(rng, 6, V, max_degree=5, with_final=True)
    graph.label[:] = np.where(rng.uniform(size=graph.num_arcs) < 0.5, V - 1, graph.label)
    _run((inputs, model, graph), 5.0, 8, 4, schedule=schedule)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_maximum_dimension(schedule):
    # C = 2,048, the largest joiner dimension (four K chunks of 512)
    rng = np.random.default_rng(22)
    V, C = 60, 2048
    model = synth.make_model(rng, V, C, 0.03)
    inputs = synth.make_inputs(rng, 3, 6, C, length_range=(4, 6))
    graph = synth.random_small_graph(rng, 8, V, max_degree=6)
    _run((inputs, model, synth.trivial_graph(V)), math.inf, 4, 4, schedule=schedule)
    _run((inputs, model, graph), 4.0, 12, 6, schedule=schedule)


def test_heavy_tailed_states():
    # one state with 5,000 arcs next to ordinary ones, as in the power-law graph's tail
    rng = np.random.default_rng(6)
    V, C, S = 60, 32, 40
    deg = rng.integers(1, 6, S)
    deg[[0, 7]] = [5000, 1200]
    g = synth._csr_from_degrees(rng, deg, V)
    g.dest[:] = np.where(rng.uniform(size=g.num_arcs) < 0.5, 0, g.dest)  # revisit state 0 often
    model = synth.make_model(rng, V, C, 0.3)
    inputs = synth.make_inputs(rng, 4, 20, C)
    _run((inputs, model, g), 6.0, 64, 16)


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_max_states_limit(schedule):
    rng = np.random.default_rng(8)
    V, C = 40, 16
    model = synth.make_model(rng, V, C, 0.5)
    inputs = synth.make_inputs(rng, 2, 15, C)
    graph = synth.random_small_graph(rng, 30, V, max_degree=10)
    _run((inputs, model, graph), math.inf, 256, 256, schedule=schedule)
    _run((inputs, model, graph), math.inf, 256, 7, schedule=schedule)


@pytest.mark.parametrize("schedule", SCHEDULES + ["stream1"])
def test_standard(schedule):
    # oracle margins: 76% of the frames precede their stream's first contested frame
    # (18 of 32 streams clean), 99.7% of the frames have a margin above 1e-4
    _, _, rep = _run("standard", math.inf, 4, 4, schedule=schedule, exact_floor=0.98)
    assert rep.streams == 32
    assert rep.frames_prefix >= 0.70 * rep.frames and rep.clean >= 14


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_graph(schedule):
    # oracle margins: 54% prefix (7 of 32 streams clean), 99.2% of frames above 1e-4
    _, _, rep = _run("graph", 4.0, 32, 8, schedule=schedule, exact_floor=0.97)
    assert rep.streams == 32
    assert rep.frames_prefix >= 0.50 * rep.frames and rep.clean >= 5


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_throughput_sampled(schedule):
    # full B = 256 on the GPU (the configuration the benchmark times), 64 streams checked;
    # bf16 margins of 2e-3 leave 94% of their frames above the threshold
    _, _, rep = _run("throughput", math.inf, 4, 4, dtype="bf16", streams=range(0, 256, 4),
                     schedule=schedule, exact_floor=0.90)
    assert rep.streams == 64


@pytest.mark.parametrize("B", [256, 1024])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_trivial_wide_frame_joiner(dtype, B):
    # trivial graph on the frame schedule with enough joiner rows (B streams, 8 contexts)
    # and columns (V = 2,000) for the 64 x 128 GEMM tiles' top-label epilogue: B = 256 gives
    # two tiles per CU, the fewest that run them, B = 1,024 eight
    rng = np.random.default_rng(11)
    model = synth.make_model(rng, 2000, 256, 0.05)
    inputs = synth.make_inputs(rng, B, 6, 256, length_range=(0, 6))
    _run((inputs, model, synth.trivial_graph(2000)), math.inf, 8, 8, dtype=dtype,
         streams=range(0, B, B // 8), schedule="frame")


@pytest.mark.parametrize("B,V", [(1500, 600), (4500, 600), (4500, 100)])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_very_wide_batch_packed_rows(dtype, B, V):
    # several streams per thread in the row packing of the 64 x 128 tiles (V = 600; 6, and 18
    # of which 16 are held) and of the sweep (V = 100; 9, 4 held), ragged so that rows shift
    rng = np.random.default_rng(B + V)
    model = synth.make_model(rng, V, 100, 0.1)
    inputs = synth.make_inputs(rng, B, 5, 100, length_range=(0, 5))
    _run((inputs, model, synth.trivial_graph(V)), math.inf, 8, 8, dtype=dtype,
         streams=list(range(0, B, B // 9)) + [B - 1], schedule="frame")


def test_general_graph_wide_batch():
    # general graph on the frame schedule with B = 1,024 streams: four search workgroups
    # per CU over the batch, two of them resident on a CU at a time (each allocates the
    # next encoder frame up to Kpad only), up to 32 x 40 candidates per stream (the hash
    # merge beyond 512); 64 streams spread over the batch checked
    rng = np.random.default_rng(21)
    V, C = 200, 64
    model = synth.make_model(rng, V, C, 0.4)
    inputs = synth.make_inputs(rng, 1024, 6, C, length_range=(0, 6))
    graph = synth.random_small_graph(rng, 40, V, max_degree=40, with_final=True)
    _, _, rep = _run((inputs, model, graph), 4.0, 32, 8, streams=range(0, 1024, 16),
                     schedule="frame")
    assert rep.streams == 64


LARGE_STREAMS = list(range(0, 128, 8))
# oracle margins on these streams: fp32 99.6% of frames above 1e-4 (58% prefix, 5 clean
# streams); bf16 91.9% above 2e-3 (4% prefix, no clean stream: the replay carries it)
LARGE_FLOOR = {"fp32": 0.97, "bf16": 0.85}


def test_large_sampled():
    # full B = 128 on the GPU, V = 5,000 and the 1M-state power-law graph; 16 streams
    # spread over the batch checked on every frame
    _, _, rep = _run("large", 8.0, 64, 16, streams=LARGE_STREAMS, exact_floor=LARGE_FLOOR["fp32"])
    assert rep.streams == 16


def test_large_bf16_sampled():
    # the Large workload with the bf16 joiner (the benchmark's large-bf16 line), the same
    # 16 streams, against the bf16-operand oracle
    _, _, rep = _run("large", 8.0, 64, 16, dtype="bf16", streams=LARGE_STREAMS,
                     exact_floor=LARGE_FLOOR["bf16"])
    assert rep.streams == 16


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_deterministic(schedule):
    w, inputs, model, graph = synth.make_workload("graph")
    from paper_2211_00484_amd import tbs
    m, gr = tbs.Model.from_synth(model), tbs.Graph.from_synth(graph)
    a = gpu_decode(model, graph, inputs, 4.0, 32, 8, model=m, graph=gr, schedule=schedule)
    b = gpu_decode(model, graph, inputs, 4.0, 32, 8, model=m, graph=gr, schedule=schedule)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


def test_schedules_agree_on_clean_streams():
    # Both schedules on one model: identical survivor traces up to each stream's first
    # frame with a decision margin <= 1e-4 (oracle), and identical results on streams
    # without one.
    w, inputs, model, graph = synth.make_workload("graph")
    from paper_2211_00484_amd import tbs
    m, gr = tbs.Model.from_synth(model), tbs.Graph.from_synth(graph)
    a = gpu_decode(model, graph, inputs, 4.0, 32, 8, model=m, graph=gr, schedule="frame")
    b = gpu_decode(model, graph, inputs, 4.0, 32, 8, model=m, graph=gr, schedule="stream")
    o = oracle.decode(model, graph, inputs.encoder_out, inputs.lengths, 4.0, 32, 8)
    fm = o.frame_margins
    compared = 0
    for s in range(inputs.B):
        L = int(inputs.lengths[s])
        bad = [t for t in range(L) if fm[s, t] <= 1e-4]
        t_star = bad[0] if bad else L
        assert np.array_equal(a["trace"][: t_star + 1, s], b["trace"][: t_star + 1, s]), s
        compared += t_star
        if not bad and fm[s, inputs.T] > 1e-4:
            assert np.array_equal(a["tokens"][s], b["tokens"][s]), s
            assert abs(a["scores"][s] - b["scores"][s]) <= 1e-4, s
    say(f"  {compared} of {int(inputs.lengths.sum())} frames compared")
    assert compared >= inputs.lengths.sum() // 2


def test_stream_schedule_refuses_what_it_cannot_hold():
    import torch
    from paper_2211_00484_amd import tbs
    rng = np.random.default_rng(4)
    model_np = synth.make_model(rng, 40, 32, 0.3)
    inputs = synth.make_inputs(rng, 2, 6, 32)
    graph_np = synth.random_small_graph(rng, 10, 40, max_degree=6)
    model = tbs.Model.from_synth(model_np)
    graph = tbs.Graph.from_synth(graph_np)
    enc = torch.from_numpy(inputs.encoder_out).cuda()
    model.set_schedule("stream")
    with pytest.raises(tbs.TbsError, match="EUNSUPPORTED"):   # 32 joiner rows per stream
        tbs.decode(model, graph, enc, inputs.lengths, max_states=32, max_contexts=32)
    model.set_schedule("auto")                                # falls back to the frame kernels
    out = tbs.decode(model, graph, enc, inputs.lengths, max_states=32, max_contexts=32)
    torch.cuda.synchronize()
    assert out.num_tokens.cpu().numpy().max() <= 6
    with pytest.raises(tbs.TbsError, match="EINVAL"):
        tbs._check(tbs.lib().tbs_model_set_schedule(model._h, 7))


def test_zero_batch_and_zero_frames():
    import torch
    from paper_2211_00484_amd import tbs
    model = tbs.Model.from_synth(synth.make_model(np.random.default_rng(0), 8, 16, 0.1))
    graph = tbs.Graph.trivial(8)
    out = tbs.decode(model, graph, torch.zeros((0, 5, 16), device="cuda"), np.zeros(0, np.int32))
    assert out.tokens.shape == (0, 5)
    out = tbs.decode(model, graph, torch.zeros((3, 0, 16), device="cuda"), np.zeros(3, np.int32),
                     want_arcs=True, want_trace=True)
    torch.cuda.synchronize()
    assert out.num_tokens.cpu().tolist() == [0, 0, 0]
    assert out.scores.cpu().tolist() == [0.0, 0.0, 0.0]


def test_invalid_arguments_rejected():
    import torch
    from paper_2211_00484_amd import tbs
    model = tbs.Model.from_synth(synth.make_model(np.random.default_rng(0), 8, 16, 0.1))
    graph = tbs.Graph.trivial(8)
    enc = torch.zeros((2, 5, 16), device="cuda")
    with pytest.raises(tbs.TbsError, match="EINVAL"):
        tbs.decode(model, graph, enc, np.array([6, 1], np.int32))
    with pytest.raises(tbs.TbsError, match="EINVAL"):
        tbs.decode(model, graph, enc, np.array([1, 1], np.int32), max_states=0)
    with pytest.raises(tbs.TbsError, match="ECAPACITY"):
        tbs.decode(model, graph, enc, np.array([1, 1], np.int32), max_states=257)
    with pytest.raises(tbs.TbsError, match="EINVAL"):
        tbs.decode(model, tbs.Graph.trivial(9), enc, np.array([1, 1], np.int32))
    with pytest.raises(tbs.TbsError, match="EINVAL"):
        tbs.decode(model, graph, enc, np.array([1, 1], np.int32), beam=-1.0)


def test_frame_loop_graph_replays_match_eager():
    # The frame schedule's loop is captured in a HIP graph the second time a decode's
    # launch arguments repeat, then replayed.  Every decode (direct, capturing, replays,
    # and after a decode with other inputs) must equal the same decode on a model with
    # capture off, with host synchronisation and eager work between the replays.
    import torch
    from paper_2211_00484_amd import tbs
    w, inputs, model_np, graph_np = synth.make_workload("graph")
    rng = np.random.default_rng(77)
    enc_np2 = rng.standard_normal(inputs.encoder_out.shape).astype(np.float32)
    lens2 = rng.integers(1, inputs.T + 1, inputs.B).astype(np.int32)
    for b in range(inputs.B):
        enc_np2[b, lens2[b]:] = 0.0
    graph = tbs.Graph.from_synth(graph_np)
    cap, ref = tbs.Model.from_synth(model_np), tbs.Model.from_synth(model_np)
    for m in (cap, ref):
        m.set_schedule("frame")
    ref.set_graph_capture(False)
    B, T = inputs.B, inputs.T
    encs = {"x": (torch.from_numpy(inputs.encoder_out).cuda(), inputs.lengths),
            "y": (torch.from_numpy(enc_np2).cuda(), lens2)}

    def run(model, which, out):
        enc, lens = encs[which]
        tbs.decode_into(model, graph, enc, lens, 4.0, 32, 8, out)
        torch.cuda.synchronize()
        return {k: getattr(out, k).cpu().numpy().copy()
                for k in ("tokens", "num_tokens", "scores", "status", "arcs", "trace")}

    mk = lambda: tbs.allocate_outputs(B, T, 32, status=True, arcs=True, trace=True)
    want = {k: run(ref, k, mk()) for k in encs}
    out = mk()
    for i, which in enumerate(["x", "x", "x", "x", "y", "x", "x", "y", "y", "y"]):
        got = run(cap, which, out)
        torch.zeros(1 << 20, device="cuda").add_(1.0)   # eager work between replays
        for k in got:
            assert np.array_equal(got[k], want[which][k]), (i, which, k)
    captures, replays = cap.graph_stats()
    say(f"  frame-loop graph: {captures} captures, {replays} replays")
    assert (captures, replays) == (2, 6)   # x: direct, capture, 2 replays; y direct; x 2 replays; y capture, 2 replays
    assert ref.graph_stats() == (0, 0)


def _tied_case(kind, seed=77):
    # Zero joiner weights and bias and zero arc scores: every label has the same
    # log-probability, so all candidates of a frame score exactly alike, in fp32 on the
    # GPU and in fp64 in the oracle, and every selection (merge, max-states, context
    # ranking, final pick) is decided by the tie-break orders alone.
    rng = np.random.default_rng(seed)
    V, C = 12, 16
    model = synth.make_model(rng, V, C, 0.3)
    model.w_out[:] = 0.0
    model.b_out[:] = 0.0
    inputs = synth.make_inputs(rng, 4, 30, C, length_range=(5, 30))
    if kind == "graph":
        graph = synth.random_small_graph(rng, 40, V, max_degree=6)
        graph.score[:] = 0.0
    else:
        graph = synth.trivial_graph(V)
    return inputs, model, graph


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("kind,beam,Ns,Nc", [("graph", math.inf, 8, 3), ("graph", 1.0, 40, 6),
                                             ("graph", math.inf, 100, 20), ("graph", 0.5, 200, 64),
                                             ("trivial", math.inf, 8, 3), ("trivial", math.inf, 4, 4)])
def test_exact_ties_follow_the_canonical_orders(kind, beam, Ns, Nc, schedule):
    from paper_2211_00484_amd import tbs
    inputs, model, graph = _tied_case(kind)
    say(f"tied decode {kind} beam={beam} Ns={Ns} Nc={Nc} {schedule}")
    try:
        g = gpu_decode(model, graph, inputs, beam, Ns, Nc, schedule=schedule)
    except tbs.TbsError as e:
        if schedule == "stream" and e.status == -5:
            pytest.skip(f"not supported by the per-stream kernel: {e}")
        raise
    streams = list(range(inputs.B))
    o = oracle.decode(model, graph, inputs.encoder_out, inputs.lengths, beam, Ns, Nc,
                      streams=streams)
    assert (o.frame_margins[:, :-1] == 0).any(), "the case has no tied decision"
    for b in streams:
        L = int(inputs.lengths[b])
        assert np.array_equal(g["trace"][: L + 1, b], o.trace[: L + 1, b]), f"stream {b}: trace"
        n = int(g["ntok"][b])
        assert g["tokens"][b, :n].tolist() == o.tokens[b, : o.ntok[b]].tolist(), f"stream {b}: tokens"
        assert int(g["status"][b]) == int(o.status[b])
        assert np.array_equal(g["arcs"][b, :L], o.arcs[b, :L]), f"stream {b}: arcs"
        assert abs(float(g["scores"][b]) - float(o.scores[b])) <= 1e-4
