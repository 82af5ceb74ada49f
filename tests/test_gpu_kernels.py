"""Single kernels at the sizes where they can go wrong (tile edges, remainders, the ends of a dispatch rule's ranges),
through graphs of one operator or a few, against float64 arithmetic on the same (rounded) operands."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2403_00176_amd as S
    return S


def run_graph(graph, sym, weights, inputs, sessions=None):
    """One run of a graph in a session of its own; the outputs as float64 arrays."""
    import torch
    from paper_2403_00176_amd.session import Session, to_host
    ses = Session(graph)
    ses.upload_weights(weights)
    b = ses.bind(sym)
    outs = ses.alloc_outputs(ses.output_shapes(b))
    ses.run(b, ses.upload_inputs(inputs), outs)
    torch.cuda.synchronize()
    return [to_host(o) for o in outs]


# fp32 contractions: a wave per column for 1, 2 and up to 4 rows (k of one chunk per lane and of more, columns that are no
# multiple of 4), 16 x 16 tiles with k split over 8 waves (rows and columns of one tile and one more, k shorter than one
# chunk per wave, k not a multiple of 4, k longer than one round of loads; few rows of many columns), 32 x 32 tiles, 64 x
# 64 FMA tiles (also where the k of a full chip is short)
@pytest.mark.parametrize("M,N,K,trans_b,batch", [
    (2, 64, 768, 1, 1), (8, 1, 64, 1, 1), (16, 16, 16, 1, 1), (17, 15, 77, 0, 3), (77, 77, 64, 1, 4), (77, 64, 77, 0, 4),
    (33, 47, 1030, 1, 1), (128, 1024, 256, 1, 1), (513, 545, 260, 1, 1), (300, 300, 131, 0, 4), (1473, 1409, 40, 1, 1),
    (1, 101, 256, 1, 1), (1, 99, 1300, 1, 1), (2, 33, 260, 1, 1), (3, 50, 256, 1, 1), (3, 50, 1028, 1, 1), (4, 7, 64, 1, 1),
    (6, 17000, 64, 1, 1), (16, 17000, 24, 1, 1), (16, 17000, 128, 1, 1), (385, 383, 68, 1, 1), (690, 1200, 140, 1, 1), (1000, 1100, 64, 1, 1)])
def test_fp32_contraction(S, M, N, K, trans_b, batch):
    from workloads import GraphBuilder
    print(f"case M {M} N {N} K {K} transB {trans_b} batch {batch}", flush=True)
    rs = np.random.RandomState(M + N + K)
    lead = [batch] if batch > 1 else []
    gb = GraphBuilder([("M", 1, 2048)])
    x = gb.input("x", "f32", lead + ["M", K])
    w = gb.weight("w", "f32", (lead if not trans_b else []) + ([N, K] if trans_b else [K, N]))
    bias, res = gb.weight("b", "f32", [N]), gb.input("r", "f32", lead + ["M", N])
    y = gb.op("Add", [gb.op("MatMul", [x, w], transB=trans_b), bias])
    gb.mark_output(gb.op("Relu", [gb.op("Add", [y, res])]), "y")
    f32 = lambda *s: rs.randn(*s).astype(np.float32).astype(np.float64)  # noqa: E731
    X, W, B, Rs = f32(*lead, M, K), f32(*((lead if not trans_b else []) + ([N, K] if trans_b else [K, N]))), f32(N), f32(*lead, M, N)
    got = run_graph(gb.build(), {"M": M}, {w: W, bias: B}, {x: X, res: Rs})[0]
    Wt = np.swapaxes(W, -1, -2) if trans_b else W
    ref = np.maximum(X @ Wt + B + Rs, 0)
    # K products and the two additions, each rounded once, in any order: (K + 3) half-ulps of the sum of magnitudes
    bound = (K + 3) * 2.0 ** -24 * (np.abs(X) @ np.abs(Wt) + np.abs(B) + np.abs(Rs))
    assert got.shape == ref.shape and (np.abs(got - ref) <= bound).all(), np.max(np.abs(got - ref) / bound)


# The plain FMA kernel is one version for every shape: the forced version 3 and a plan without multi-version kernels give
# the same bits, where the automatic choice splits k and so sums in another order.
@pytest.mark.parametrize("M,K", [(2, 768), (77, 1024)])
def test_fp32_plain_version(S, M, K):
    import torch
    from paper_2403_00176_amd.session import Session
    from workloads import GraphBuilder
    rs = np.random.RandomState(M)
    X, W, got = rs.randn(M, K), rs.randn(256, K), {}
    for how in ("automatic", "forced", "one version"):
        gb = GraphBuilder([("M", 1, 2048)])
        x, w = gb.input("x", "f32", ["M", K]), gb.weight("w", "f32", [256, K])
        gb.mark_output(gb.op("MatMul", [x, w], transB=1), "y")
        ses = Session(gb.build(), mvc=0 if how == "one version" else 1)
        ses.upload_weights({w: W})
        b = ses.bind({"M": M})
        S.sod2_binding_force_variant(b, 3 if how == "forced" else -1)
        outs = ses.alloc_outputs(ses.output_shapes(b))
        ses.run(b, ses.upload_inputs({x: X}), outs)
        torch.cuda.synchronize()
        got[how] = outs[0]
    assert torch.equal(got["forced"], got["one version"]) and not torch.equal(got["forced"], got["automatic"])


# A contraction whose first operand repeats one row (an Expand: row stride 0), plain (with k split over workgroups) and
# with the LayerNorm behind it folded into it and into the contraction that reads it.
@pytest.mark.parametrize("M,K,folded", [(512, 256, True), (333, 768, True), (64, 4096, False)])
def test_contraction_of_a_broadcast_row(S, M, K, folded):
    import torch
    from paper_2403_00176_amd.session import Session, to_host
    from workloads import GraphBuilder
    print(f"case M {M} K {K} folded {folded}", flush=True)
    N, N2 = 512, 320
    rs = np.random.RandomState(M + K)
    bf = lambda *s: torch.from_numpy(rs.randn(*s).astype(np.float32)).bfloat16().double().numpy()  # noqa: E731
    gb = GraphBuilder([("M", 1, 2048)])
    x, like = gb.input("x", "bf16", [1, K]), gb.input("like", "bf16", ["M", K])
    w, b = gb.weight("w", "bf16", [N, K]), gb.weight("b", "bf16", [N])
    y = gb.op("Add", [gb.op("MatMul", [gb.op("Expand", [x, gb.op("Shape", [like], dtype="i64")]), w], transB=1), b])
    X, W, B = bf(1, K), bf(N, K) / 16, bf(N)
    weights, mid = {w: W, b: B}, X @ W.T + B
    if folded:
        gm, bt, w2 = gb.weight("gm", "bf16", [N]), gb.weight("bt", "bf16", [N]), gb.weight("w2", "bf16", [N2, N])
        gb.mark_output(gb.op("MatMul", [gb.op("LayerNorm", [y, gm, bt], eps=1e-5), w2], transB=1), "z")
        G, T, W2 = bf(N), bf(N), bf(N2, N) / 16
        weights.update({gm: G, bt: T, w2: W2})
        rstd = 1 / np.sqrt(mid.var() + 1e-5)
        norm = (mid - mid.mean()) * rstd * G
        ref = (norm + T) @ W2.T
        # bf16 roundings on the way: the first result (which may also land on the neighbouring value), its product with
        # the scale, the result; half an ulp is 2^-9 of the value
        bound = (2.0 ** -8 + 2.0 ** -9) * (np.abs(mid * rstd * G) @ np.abs(W2.T)) + 2.0 ** -8 * (np.abs(ref) + np.abs(T) @ np.abs(W2.T))
    else:
        gb.mark_output(y, "z")
        ref, bound = mid, 2.0 ** -8 * np.abs(mid) + 2.0 ** -18 * (np.abs(X) @ np.abs(W.T) + np.abs(B))
    ses = Session(gb.build())
    ses.upload_weights(weights)
    bnd = ses.bind({"M": M})
    outs = ses.alloc_outputs(ses.output_shapes(bnd))
    arena = ses.ensure_arena(S.sod2_binding_arena_bytes(bnd)[0])
    arena.fill_(0xff)                                          # (NaN wherever nothing is written)
    ses.run(bnd, ses.upload_inputs({x: X, like: np.zeros((M, K))}), outs)
    torch.cuda.synchronize()
    trace = [e for e in S.sod2_run_trace(bnd) if e["is_group"]]
    assert [e["fold"] for e in trace] == ([1, 2] if folded else [0])
    assert folded or trace[0]["splits"] > 1
    got = to_host(outs[0])
    assert got.shape == (M, ref.shape[1]) and (np.abs(got - ref) <= bound).all(), np.max(np.abs(got - ref) / bound)


STEP = 23                                          # kernel of a trace entry: a phase of a step that ran as one kernel


def cache_offsets(S, desc, binding):
    """Where the cached keys and values of every layer lie: the session slots of the CacheAppend results."""
    at = [S.sod2_binding_query_tensor(binding, op.outputs[0]) for op in desc.ops if op.kind == "CacheAppend"]
    assert all(i["where"] == "session" for i in at) and len({i["offset"] for i in at}) == len(at) == len(desc.session_inputs())
    return [i["offset"] for i in at]


def ran_as_one_kernel(S, binding):
    kernels = {e["kernel"] for e in S.sod2_run_trace(binding)}
    assert kernels == {STEP} or STEP not in kernels
    return kernels == {STEP}


# The decode step as one kernel against the same launches one by one: widths whose rows deal out in whole pairs to 256,
# 192, 256, 256, 192, 128 and 64 workgroups (of a chip with 256 CUs) and one, 640, that no number of them suits; cache
# lengths at the edges of the parts of 128 keys an attention workgroup takes, one and many parts.
@pytest.mark.parametrize("hidden,heads,ffn,vocab,P", [(512, 8, 1024, 1000, 126), (768, 12, 3072, 2002, 1), (1024, 16, 4096, 32000, 383),
                                                      (512, 8, 2560, 998, 511), (768, 12, 1536, 5000, 250), (256, 4, 1024, 3000, 129),
                                                      (128, 2, 512, 200, 300), (640, 10, 2560, 1000, 64)])
def test_decode_step_as_one_kernel(S, hidden, heads, ffn, vocab, P):
    import torch
    from paper_2403_00176_amd.session import DecoderSession
    from workloads import configs
    print(f"case hidden {hidden} heads {heads} ffn {ffn} vocab {vocab} P {P}", flush=True)
    steps = 6
    w = configs.decoder(layers=2, hidden=hidden, heads=heads, ffn=ffn, vocab=vocab, p_range=(1, 512), t_max=steps + 2, n_prompts=1)
    ses = DecoderSession(w.prefill, w.decode, w.t_max)
    ses.upload_weights(w.make_weights_by_name())
    ses.start(P, vocab)
    ses.prefill(torch.from_numpy(np.random.RandomState(P).randint(0, vocab, P)).to(ses.device))
    forced = torch.from_numpy(np.random.RandomState(P + 1).randint(0, vocab, steps)).to(ses.device)
    torch.cuda.synchronize()

    def run(one_by_one):
        for t in range(steps):
            with torch.cuda.stream(ses.stream):
                ses.tokens[P + t] = forced[t]                    # teacher forcing: both paths see the same tokens
            b = ses.dec.bind({"P": P, "t": t})
            if one_by_one:
                S.sod2_binding_force_variant(b, 6)
            ses.decode(t, b)
            assert ran_as_one_kernel(S, b) == (not one_by_one and hidden != 640)
        torch.cuda.synchronize()
        d = w.decode
        caches = [ses.arena[at:at + (P + steps) * hidden * 2].view(torch.bfloat16).float().clone()
                  for at in cache_offsets(S, d, b)]
        return ses.logits[1:steps + 1].float().clone(), ses.tokens[P + 1:P + steps + 1].clone(), caches

    ref, one = run(True), run(False)
    # both round every operator's row to bf16, sums in another order: a value next to a rounding boundary may fall on
    # either side (2^-8), and passes through at most 10 more roundings of its own size: far below the 2e-2 of the oracle
    for a, b in [(ref[0], one[0])] + list(zip(ref[2], one[2])):
        assert torch.isfinite(b).all()
        assert ((a - b).norm() / a.norm()).item() <= 2 ** -8, ((a - b).norm() / a.norm()).item()
    # the token behind the last step is the arg-max of that step's logits, the lowest index among equals
    last = one[0][steps - 1]
    assert int(one[1][steps - 1]) == int((last == last.max()).nonzero()[0])
    # the same steps as a replay, bit for bit
    ses.logits.zero_()
    with torch.cuda.stream(ses.stream):
        ses.tokens[P] = forced[0]
    ses.decode(0)
    torch.cuda.synchronize()
    row = ses.logits[1].clone()
    ses.decode_replay(0, 1)
    assert S.sod2_replay_one_kernel(ses.replay) == (hidden != 640)
    torch.cuda.synchronize()
    assert torch.equal(row, ses.logits[1])


# A binding that forces a version or a number of k ranges, or that is profiled, runs its groups one by one.
def test_forced_and_profiled_decode_steps_run_group_by_group(S):
    import torch
    from paper_2403_00176_amd.session import DecoderSession
    from workloads import configs
    w = configs.decoder(layers=2, hidden=256, heads=4, ffn=512, vocab=200, p_range=(1, 512), t_max=4, n_prompts=1)
    ses = DecoderSession(w.prefill, w.decode, w.t_max)
    ses.upload_weights(w.make_weights_by_name())
    ses.start(20, 200)
    ses.prefill(torch.arange(20).to(ses.device))
    for force, one in [(lambda b: None, True), (lambda b: S.sod2_binding_force_variant(b, 6), False),
                       (lambda b: S.sod2_binding_force_splits(b, 2), False), (lambda b: S.sod2_binding_set_profiling(b, True), False)]:
        b = ses.dec.bind({"P": 20, "t": 0})
        force(b)
        ses.decode(0, b)
        assert ran_as_one_kernel(S, b) == one
    torch.cuda.synchronize()


# A plan without multi-version kernels has one version of every contraction: neither its runs nor its replays are one kernel.
def test_decode_step_of_a_plan_of_one_version(S):
    import torch
    from paper_2403_00176_amd.session import DecoderSession
    from workloads import configs
    w = configs.decoder(layers=2, hidden=256, heads=4, ffn=512, vocab=200, p_range=(1, 512), t_max=4, n_prompts=1)
    ses = DecoderSession(w.prefill, w.decode, w.t_max, mvc=0)
    ses.upload_weights(w.make_weights_by_name())
    ses.start(20, 200)
    ses.prefill(torch.arange(20).to(ses.device))
    assert not ran_as_one_kernel(S, ses.decode(0))
    d = w.decode
    fixed = [0] * len(d.inputs()), [0] * len(d.outputs())      # (nothing that moves: only skinny contractions follow a moving result)
    ins = {"ids": ses.tokens[20:], "pos": ses.positions[20:]}
    outs = {"logits": ses.logits[1], "next": ses.tokens[21:]}
    replay = S.sod2_replay_create(ses.dec.plan, {"P": 20, "t": 0}, "t", 4, ses.arena.data_ptr(), ses.arena.numel(),
                                  [x.data_ptr() for x in ses.dec.weights], [ins[d.tensors[t].name].data_ptr() for t in d.inputs()], fixed[0],
                                  [outs[d.tensors[t].name].data_ptr() for t in d.outputs()], fixed[1], ses.step_counter.data_ptr(),
                                  ses.stream.cuda_stream)
    torch.cuda.synchronize()
    row = ses.logits[1].clone()
    ses.logits[1].zero_()
    torch.cuda.synchronize()
    S.sod2_replay_launch(replay, 0, 1, ses.stream.cuda_stream)
    assert not S.sod2_replay_one_kernel(replay)
    torch.cuda.synchronize()
    assert torch.equal(row, ses.logits[1])


# The null stream takes the one-kernel step like any other stream of the device.
def test_decode_step_on_the_null_stream(S):
    import torch
    from paper_2403_00176_amd.session import DecoderSession
    from workloads import configs
    w = configs.decoder(layers=2, hidden=256, heads=4, ffn=512, vocab=200, p_range=(1, 512), t_max=4, n_prompts=1)
    ses = DecoderSession(w.prefill, w.decode, w.t_max)
    ses.upload_weights(w.make_weights_by_name())
    ses.start(20, 200)
    ses.prefill(torch.arange(20).to(ses.device))
    ses.decode(0)
    torch.cuda.synchronize()
    row = ses.logits[1].clone()
    ses.logits[1].zero_()
    torch.cuda.synchronize()
    ses.stream = ses.dec.stream = torch.cuda.default_stream()
    assert ses.stream.cuda_stream == 0
    assert ran_as_one_kernel(S, ses.decode(0))
    torch.cuda.synchronize()
    assert torch.equal(row, ses.logits[1])


# A session of a device that is not the calling thread's current one: its steps run group by group (the exchange buffer
# and the step table are the current device's).
def test_decode_step_of_another_device(S):
    import torch
    from paper_2403_00176_amd.session import DecoderSession
    from workloads import configs
    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs")
    w = configs.decoder(layers=2, hidden=256, heads=4, ffn=512, vocab=200, p_range=(1, 512), t_max=4, n_prompts=1)
    logits = []
    for device in ("cuda:0", "cuda:1"):
        ses = DecoderSession(w.prefill, w.decode, w.t_max, device=device)
        ses.upload_weights(w.make_weights_by_name())
        ses.start(20, 200)
        ses.prefill(torch.arange(20).to(ses.device))
        assert torch.cuda.current_device() == 0
        assert ran_as_one_kernel(S, ses.decode(0)) == (device == "cuda:0")
        torch.cuda.synchronize(ses.device)
        logits.append(ses.logits[1].float().cpu())
    assert ((logits[0] - logits[1]).norm() / logits[0].norm()).item() <= 2 ** -8


# Rows of nearly equal values whose squares overflow fp32 (1e19 and up) while the distances from their mean do not: the
# LayerNorms of the one-kernel step take the variance from the distances, like those of the launches one by one.
def test_decode_step_of_large_rows(S):
    import torch
    from paper_2403_00176_amd.session import DecoderSession
    from workloads import configs
    P, steps, vocab = 40, 3, 1000
    w = configs.decoder(layers=2, hidden=512, heads=8, ffn=1024, vocab=vocab, p_range=(1, 512), t_max=steps + 2, n_prompts=1)
    weights = w.make_weights_by_name()
    rs = np.random.RandomState(7)
    weights["tok_emb"] = 2.0 ** 64 * (1 + 2.0 ** -6 * rs.randint(0, 4, weights["tok_emb"].shape))
    ses = DecoderSession(w.prefill, w.decode, w.t_max)
    ses.upload_weights(weights)
    ses.start(P, vocab)
    ses.prefill(torch.from_numpy(rs.randint(0, vocab, P)).to(ses.device))
    forced = torch.from_numpy(rs.randint(0, vocab, steps)).to(ses.device)
    logits = []
    for variant in (6, -1):
        for t in range(steps):
            with torch.cuda.stream(ses.stream):
                ses.tokens[P + t] = forced[t]
            b = ses.dec.bind({"P": P, "t": t})
            S.sod2_binding_force_variant(b, variant)
            ses.decode(t, b)
            assert ran_as_one_kernel(S, b) == (variant == -1)
        torch.cuda.synchronize()
        logits.append(ses.logits[1:steps + 1].double())
    a, b = logits
    # the rows of tokens differ in their LayerNorm, so equal logits would mean that only its shift was left
    assert torch.isfinite(a).all() and (a[0] - a[1]).norm() > 0.1 * a[0].norm()
    assert ((a - b).norm() / a.norm()).item() <= 2 ** -8, ((a - b).norm() / a.norm()).item()


# Two sequences stepped in turn on two streams, nothing waited for between them: the one-kernel steps are put in order.
def test_decode_steps_of_two_streams(S):
    import torch
    from paper_2403_00176_amd.session import DecoderSession
    from workloads import configs
    steps, lengths = 6, (126, 31)
    w = configs.decoder(layers=2, hidden=512, heads=8, ffn=1024, vocab=1000, p_range=(1, 512), t_max=steps + 2, n_prompts=1)
    weights = w.make_weights_by_name()
    sessions = []
    for P in lengths:
        ses = DecoderSession(w.prefill, w.decode, w.t_max)
        ses.upload_weights(weights)
        ses.start(P, 1000)
        ses.prefill(torch.from_numpy(np.random.RandomState(P).randint(0, 1000, P)).to(ses.device))
        sessions.append(ses)
    torch.cuda.synchronize()
    assert sessions[0].stream != sessions[1].stream
    for t in range(steps):
        for ses in sessions:
            assert ran_as_one_kernel(S, ses.decode(t))
    torch.cuda.synchronize()
    together = [(s.logits.clone(), s.tokens.clone()) for s in sessions]
    for ses, (logits, tokens) in zip(sessions, together):      # each on its own, the same tokens and bits
        ses.logits[1:steps + 1].zero_()
        torch.cuda.synchronize()
        ses.decode_replay(0, steps)
        torch.cuda.synchronize()
        assert torch.equal(ses.logits[:steps + 1], logits[:steps + 1]) and torch.equal(ses.tokens, tokens)
