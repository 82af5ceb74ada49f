"""The work that users of this framework have it do, as cases that can be timed.

A pass is what a serving program does for one request: bind the plan to the shapes of the request
(every request has its own), run it on the device, leave the results in the caller's buffers.  The
models are the seven synthetic workloads of ``workloads.configs``, with random weights drawn once per
process (a model is loaded once and serves many requests); the inputs come from the seed.

The sizes span the declared ranges: batch 1..8 and 32..512 tokens for the encoder, 128..384 tokens for the
encoders that skip layers, 16..128 tokens for the fp32 block, images of 224..640 pixels (any size, not
only multiples of 32), prompts of 64..512 tokens and greedy decoding behind them.
"""
import numpy as np
import torch

import paper_2403_00176_amd as S
from paper_2403_00176_amd.session import DecoderSession, Session
from workloads import configs

DEV = "cuda:0"
HIDDEN, LAYERS, FFN = 768, 12, 3072              # the bf16 encoders
GATE_GAIN, MARK = 0.5, 6.0                       # scale of the gates' first layer, size of the marks they read


def listed():
    return [
        # one short sentence: the smallest request of a text service, all launches and latency
        {"name": "encoder B1 L32", "model": "encoder", "B": 1, "L": 32},
        # an ordinary ragged batch: nothing is a multiple of a tile
        {"name": "encoder B3 L197", "model": "encoder", "B": 3, "L": 197},
        # the largest batch of the largest length: throughput
        {"name": "encoder B8 L512", "model": "encoder", "B": 8, "L": 512},
        # full-precision block on one short sequence
        {"name": "block f32 L77", "model": "block", "L": 77},
        # image classification, the smallest image of the range
        {"name": "cnn 224x224", "model": "cnn", "H": 224, "W": 224},
        # ... and the largest
        {"name": "cnn 640x640", "model": "cnn", "H": 640, "W": 640},
        # detection neck on a camera frame that is not square and not a multiple of 32 (computed resize shapes)
        {"name": "neck 417x593", "model": "neck", "H": 417, "W": 593},
        # encoder with a skip decision per layer, read back in the middle of the run
        {"name": "gated B4 L250 run 6", "model": "gated", "B": 4, "L": 250, "kept": 6},
        # encoder with a decision per layer and sequence: compaction, re-planning in the middle of the run
        {"name": "compact B6 L207 keep 3", "model": "compact", "B": 6, "L": 207, "kept": 3},
        # prompt pass of a chat request
        {"name": "prefill P437", "model": "prefill", "P": 437},
        # greedy decoding: the steps replayed from one captured graph
        {"name": "decode replay P300 n32", "model": "decode", "P": 300, "n": 32, "replay": True},
        # ... and bound and launched one by one, as a host that looks at every token does
        {"name": "decode steps P97 n12", "model": "decode", "P": 97, "n": 12, "replay": False},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    model = rng.choice(["encoder", "encoder", "encoder", "block", "cnn", "cnn", "neck", "gated", "compact", "prefill",
                        "decode", "decode"])
    if model == "encoder":
        return {"model": model, "B": rng.randint(1, 8), "L": _log_int(rng, 32, 512)}
    if model == "block":
        return {"model": model, "L": rng.randint(16, 128)}
    if model in ("cnn", "neck"):
        if rng.random() < 0.5:                   # the multiples of 32 that detectors are fed
            return {"model": model, "H": 32 * rng.randint(7, 20), "W": 32 * rng.randint(7, 20)}
        return {"model": model, "H": rng.randint(224, 640), "W": rng.randint(224, 640)}
    if model == "gated":
        return {"model": model, "B": 4, "L": rng.randint(128, 384), "kept": rng.randint(3, 9)}
    if model == "compact":
        B = rng.randint(2, 8)
        return {"model": model, "B": B, "L": rng.randint(128, 384), "kept": rng.randint(1, B)}
    if model == "prefill":
        return {"model": model, "P": rng.randint(64, 512)}
    return {"model": model, "P": rng.randint(64, 480), "n": rng.randint(6, 30), "replay": rng.random() < 0.5}


# ---- models: one session per model and process --------------------------------------------------

_sessions = {}


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _values(spec, shape, gen):
    if spec[0] == "const":
        return np.full(shape, spec[1], np.float32)
    return torch.empty(shape, device=DEV).normal_(spec[1], spec[2], generator=gen).cpu().numpy()


def _marks():
    """One direction of the residual stream per layer, orthonormal: what the gates of the skipping encoders look at."""
    g = torch.Generator().manual_seed(77)
    q, _ = torch.linalg.qr(torch.randn(HIDDEN, LAYERS, generator=g, dtype=torch.float64))
    return q.T.float()


def _model(name):
    if name in _sessions:
        return _sessions[name]
    w = {"encoder": configs.config2, "block": configs.config1, "cnn": configs.config3, "neck": configs.config7,
         "gated": configs.config4, "compact": configs.config6}[name](n_calls=1)
    gen = _generator(1000 + sum(map(ord, name)))
    weights = {t: _values(w.weight_spec[t], tuple(w.graph.tensors[t].dims), gen) for t in w.graph.weights()}
    if name in ("gated", "compact"):
        # a trained gate is decided: its first two units read the layer's mark in the pooled activations (one for
        # either sign), the others carry noise; so a rounding does not turn a decision over
        for l, v in enumerate(_marks().numpy()):
            fc1 = weights[w.graph.tensor_id(f"g{l}.fc1.w")]
            fc1 *= 0.02 / max(float(fc1.std()), 1e-6)
            fc1[0], fc1[1] = GATE_GAIN * v, -GATE_GAIN * v
            weights[w.graph.tensor_id(f"g{l}.fc1.b")][:] = 0
            fc2 = weights[w.graph.tensor_id(f"g{l}.fc2.w")]
            fc2 *= 0.02 / max(float(fc2.std()), 1e-6)
            fc2[0, 0], fc2[0, 1] = 2.0, -2.0
            weights[w.graph.tensor_id(f"g{l}.fc2.b")][:] = 0
    ses = Session(w.graph, device=DEV)
    ses.upload_weights(weights)
    _sessions[name] = (w, ses)
    return _sessions[name]


def _decoder(P):
    """A sequence of its own (arena with the cache, tokens, logits) on the one set of decoder weights."""
    if "decoder" not in _sessions:
        w = configs.config5(n_prompts=1)
        gen = _generator(5000)
        shapes = {t.name: tuple(t.dims) for t in w.prefill.tensors if t.role == "weight"}
        by_name = {n: _values(s, shapes[n], gen) for n, s in w.weight_spec.items()}
        # A trained language model is sure of most of its tokens.  Random weights are not (the two best of 32000
        # logits are often equal in bf16, and greedy sequences part there), so the embedding dominates the
        # residual stream and the output layer looks for the embedding of a token's successor.
        emb = by_name["tok_emb"] * 50.0
        successor = np.random.RandomState(5).permutation(w.vocab)
        by_name["tok_emb"] = emb
        by_name["lm_head"] = emb[successor] * 0.02
        base = DecoderSession(w.prefill, w.decode, w.t_max, device=DEV)
        base.upload_weights(by_name)
        _sessions["decoder"] = (w, base)
    w, base = _sessions["decoder"]
    ses = DecoderSession(w.prefill, w.decode, w.t_max, device=DEV)
    ses.pre.weights = ses.dec.weights = base.pre.weights
    ses.pre.prepare_constants()
    ses.dec.prepare_constants()
    ses.start(P, w.vocab)
    return w, ses


def _cache(w, ses, binding, rows):
    """The cached keys and values of every layer: the sequence's state."""
    d, out = w.decode, []
    for t in d.session_inputs():
        at = S.sod2_binding_query_tensor(binding, t)["offset"]
        cols = d.tensors[t].dims[1]
        out.append(ses.arena[at:at + rows * cols * 2].view(torch.bfloat16).view(rows, cols))
    return out


# ---- states and passes ---------------------------------------------------------------------------

def prepare(case, seed):
    model, gen = case["model"], _generator(seed)
    if model in ("prefill", "decode"):
        w, ses = _decoder(case["P"])
        prompt = torch.randint(0, w.vocab, (case["P"],), generator=gen, device=DEV)
        state = {"case": case, "ses": ses, "prompt": prompt}
        if model == "decode":
            ses.stream.wait_stream(torch.cuda.current_stream())
            ses.prefill(prompt)                  # the cache and the first token are there
            n = case["n"]
            last = ses.dec.bind({"P": case["P"], "t": n - 1})
            state["out"] = [ses.tokens[case["P"] + 1:case["P"] + 1 + n], ses.logits[1:1 + n]] + _cache(w, ses, last, case["P"] + n)
        else:
            state["out"] = [ses.tokens[case["P"]:case["P"] + 1], ses.logits[:1]] + _cache(w, ses, ses.b_pre, case["P"])
        return state

    w, ses = _model(model)
    sym = {k: case[k] for k in ("B", "L", "H", "W") if k in case and (k != "B" or model in ("encoder", "compact"))}
    if model in ("cnn", "neck"):
        x = torch.rand((1, case["H"], case["W"], 3), generator=gen, device=DEV)
    else:
        B, L = case.get("B", 1), case["L"]
        x = torch.empty((B, L, 256 if model == "block" else HIDDEN), device=DEV).normal_(generator=gen)
        if model in ("gated", "compact"):
            # the request carries what the gates look at: the named number of layers run (or of sequences, in every layer)
            n = LAYERS if model == "gated" else B
            rows = 1 if model == "gated" else LAYERS
            order = torch.argsort(torch.rand((rows, n), generator=gen, device=DEV), dim=1)
            runs = torch.where(order < case["kept"], 1.0, -1.0)
            signs = -runs.expand(B, n) if model == "gated" else runs.T      # gated: above the threshold = skip
            x += (MARK * signs @ _marks().to(DEV))[:, None, :]
    x = x if model == "block" else x.to(torch.bfloat16)
    binding = ses.bind(sym)
    ses.ensure_arena(S.sod2_binding_arena_bytes(binding)[0])
    return {"case": case, "ses": ses, "sym": sym, "in": [x], "out": ses.alloc_outputs(ses.output_shapes(binding))}


def run(state):
    case, ses = state["case"], state["ses"]
    if case["model"] in ("prefill", "decode"):
        # the prompt comes from the caller's stream and the results are used on it: one request after the other
        ses.stream.wait_stream(torch.cuda.current_stream())
        if case["model"] == "prefill":
            ses.prefill(state["prompt"])
        elif case["replay"]:
            ses.decode_replay(0, case["n"])
        else:
            for t in range(case["n"]):
                ses.decode(t)
        torch.cuda.current_stream().wait_stream(ses.stream)
    else:
        binding = ses.bind(state["sym"])
        ses.run(binding, state["in"], state["out"])
    return state["out"]


# ---- what a pass cannot do without ---------------------------------------------------------------

def _layer(rows, keys, hidden, ffn, causal=False):
    """(flops, weight elements) of one encoder or decoder block over rows of keys tokens each."""
    n = rows * keys
    weights = 4 * hidden * hidden + 2 * hidden * ffn
    return 2 * n * weights + 4 * rows * keys * keys * hidden * (0.5 if causal else 1.0), weights


def _cnn(H, W, neck):
    flops = elements = 0

    def conv(h, w, cin, cout, k, stride=1):
        nonlocal flops, elements
        oh, ow = -(-h // stride), -(-w // stride)
        flops += 2 * oh * ow * cout * k * k * cin
        elements += cout * k * k * cin
        return oh, ow

    h, w = conv(H, W, 3, 64, 7, 2)
    h, w = -(-h // 2), -(-w // 2)
    cin, maps = 64, []
    for s, n in enumerate((3, 4, 6, 3)):
        mid, cout = 64 << s, 256 << s
        for i in range(n):
            stride = 2 if i == 0 and s > 0 else 1
            conv(h, w, cin, mid, 1)
            oh, ow = conv(h, w, mid, mid, 3, stride)
            conv(oh, ow, mid, cout, 1)
            if i == 0:
                conv(h, w, cin, cout, 1, stride)
            h, w, cin = oh, ow, cout
        maps.append((h, w, cout))
    out = 0
    if neck:
        for (h, w, c) in maps[1:]:
            conv(h, w, c, 256, 1)                # lateral
            conv(h, w, 256, 256, 1)              # head
            out += h * w * 256
        for (h, w, _) in maps[1:3]:
            conv(h, w, 512, 256, 3)              # fuse
    else:
        flops += 2 * 2048 * 1000
        elements += 2048 * 1000
        out = 1000
    return flops, elements, H * W * 3 + out


def work(case):
    model = case["model"]
    if model in ("cnn", "neck"):
        flops, weights, io = _cnn(case["H"], case["W"], model == "neck")
        return {"bytes": 2 * (weights + io), "flops": flops}
    if model == "block":
        flops, weights = _layer(1, case["L"], 256, 1024)
        return {"bytes": 4 * (weights + 2 * case["L"] * 256), "flops": flops}
    if model in ("encoder", "gated", "compact"):
        B, L = case["B"], case["L"]
        io = 2 * B * L * HIDDEN
        ran, rows = (case["kept"], B) if model == "gated" else (LAYERS, case["kept"] if model == "compact" else B)
        flops, weights = _layer(rows, L, HIDDEN, FFN)
        return {"bytes": 2 * (ran * weights + io), "flops": ran * flops}
    hidden, ffn, layers, vocab, P = 1024, 4096, 24, 32000, case["P"]
    if model == "prefill":
        flops, weights = _layer(1, P, hidden, ffn, causal=True)
        return {"bytes": 2 * (layers * (weights + 2 * P * hidden) + P * hidden + vocab * hidden + vocab),
                "flops": layers * flops + 2 * vocab * hidden}
    n, weights = case["n"], 4 * hidden * hidden + 2 * hidden * ffn
    keys = sum(P + t + 1 for t in range(n))      # every step streams the weights and the cached rows
    return {"bytes": 2 * (n * (layers * weights + vocab * (hidden + 1)) + layers * 2 * hidden * keys),
            "flops": 2 * n * (layers * weights + vocab * hidden) + layers * 4 * hidden * keys}


def tolerance(case):
    if case["model"] == "block":
        return {"rel": 1e-5}
    # bf16 storage between the operators: one rounding (2e-3 rms) per operator on the way through 12 to 24 blocks or 50
    # convolutions, each its own in another fusion; tokens are whole numbers and stay the same
    return {"rel": 1.5e-2}
