"""The waits inside a decode step that runs as one kernel, brought to their limits: the limits are lowered per binding, and
every kernel ends by itself.  (Last of the GPU tests: the final case leaves the process without that kernel.)"""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
STEP = 23                                          # kernel of a trace entry: a phase of a step that ran as one kernel
REST = 5.2                                         # seconds after which the kernel is used again (5, and some)


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2403_00176_amd as S
    return S


class Sequence:
    """A small decoder behind a prompt of P tokens, stepped with given tokens."""

    def __init__(self, S, hidden, heads, ffn, vocab, P, steps):
        import torch
        from paper_2403_00176_amd.session import DecoderSession
        from workloads import configs
        self.S, self.P, self.steps, self.hidden = S, P, steps, hidden
        self.w = configs.decoder(layers=2, hidden=hidden, heads=heads, ffn=ffn, vocab=vocab, p_range=(1, 512), t_max=steps + 2, n_prompts=1)
        self.ses = DecoderSession(self.w.prefill, self.w.decode, self.w.t_max)
        self.ses.upload_weights(self.w.make_weights_by_name())
        self.ses.start(P, vocab)
        self.ses.prefill(torch.from_numpy(np.random.RandomState(P).randint(0, vocab, P)).to(self.ses.device))
        self.forced = torch.from_numpy(np.random.RandomState(P + 1).randint(0, vocab, steps)).to(self.ses.device)
        torch.cuda.synchronize()

    def step(self, t, variant=-1, **waits):
        """Step t; whether it was one kernel."""
        import torch
        with torch.cuda.stream(self.ses.stream):
            self.ses.tokens[self.P + t] = self.forced[t]
        b = self.ses.dec.bind({"P": self.P, "t": t})
        self.S.sod2_binding_force_variant(b, variant)
        if waits:
            self.S.sod2_binding_force_waits(b, **waits)
        self.ses.decode(t, b)
        self.last = b
        return {e["kernel"] for e in self.S.sod2_run_trace(b)} == {STEP}

    def state(self):
        """Logits and cache rows of the steps."""
        import torch
        torch.cuda.synchronize()
        n = self.P + self.steps
        cache = [self.ses.arena[at:at + n * self.hidden * 2].view(torch.bfloat16).double().clone()
                 for at in (self.S.sod2_binding_query_tensor(self.last, op.outputs[0])["offset"]       # (the session slots)
                            for op in self.w.decode.ops if op.kind == "CacheAppend")]
        assert len(cache) == 4
        return self.ses.logits[1:self.steps + 1].double().clone(), cache


# Both ways round 17 rows to bf16 from the embedding to the logits of two layers (7 per layer, the embedding, the last
# LayerNorm, the logits), sums in another order: at most 2^-9 of the value each, 2^-9 / sqrt(3) in the mean square, and no
# more than if the roundings of the two had nothing to do with one another.
BAR = (2 * 17 / 3) ** 0.5 * 2.0 ** -9


def distance(a, b):
    return ((a - b).norm() / a.norm()).item()


def same(got, ref):
    import torch
    for a, b in [(ref[0], got[0])] + list(zip(ref[1], got[1])):
        assert torch.isfinite(b).all() and distance(a, b) <= BAR, distance(a, b)


# One workgroup does the whole step (the others were not waited for): widths, cache lengths at the edges of its blocks of
# 8 keys and of one wave's share of the heads; the host then leaves the kernel alone for a while and comes back to it.  (Every test leaves it in use, but the last.)
@pytest.mark.parametrize("hidden,heads,ffn,vocab,P", [(512, 8, 1024, 1000, 126), (768, 12, 3072, 2002, 1), (1024, 16, 4096, 32000, 383),
                                                      (256, 4, 1024, 3000, 8)])
def test_step_done_by_one_workgroup(S, hidden, heads, ffn, vocab, P):
    import torch
    print(f"case hidden {hidden} heads {heads} ffn {ffn} vocab {vocab} P {P}", flush=True)
    seq = Sequence(S, hidden, heads, ffn, vocab, P, 3)
    for t in range(3):
        assert not seq.step(t, variant=6)
    ref = seq.state()
    seq.ses.logits.zero_()
    torch.cuda.synchronize()
    assert seq.step(0, arrive_us=0)
    torch.cuda.synchronize()
    first = seq.ses.logits[1].float()
    assert int(seq.ses.tokens[P + 1]) == int((first == first.max()).nonzero()[0])
    assert not seq.step(1)                         # (reads the cache rows the lone workgroup wrote)
    assert not seq.step(2)
    same(seq.state(), ref)
    # a replay made meanwhile does the same: launches of its graph now, one kernel per step later
    seq.ses.decode_replay(0, 1)
    assert not S.sod2_replay_one_kernel(seq.ses.replay)
    torch.cuda.synchronize()
    row = seq.ses.logits[1].double().clone()
    time.sleep(REST)
    seq.ses.decode_replay(0, 1)
    assert S.sod2_replay_one_kernel(seq.ses.replay)
    torch.cuda.synchronize()
    assert distance(row, seq.ses.logits[1].double()) <= BAR


# A step while a kernel of another stream holds one or two CUs for some milliseconds: the workgroups that start wait for the
# others, call the exchange off, and the last to come does the step.  (Streams may share a hardware queue, behind which the
# step would simply wait its turn: several are tried.)
def test_step_beside_a_kernel_that_holds_a_cu(S):
    import torch
    seq = Sequence(S, 512, 8, 1024, 1000, 60, 8)
    for t in range(8):
        seq.step(t, variant=6)
    ref = seq.state()
    seq.ses.logits.zero_()
    rows = torch.randn(2, 1 << 23, device="cuda:0")
    streams = [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()
    called_off = 0
    for k, side in enumerate(streams):
        with torch.cuda.stream(side):
            torch.cumsum(rows, 1)                  # a row to a workgroup
        assert seq.step(2 * k, arrive_us=100)
        torch.cuda.synchronize()
        off = not seq.step(2 * k + 1)
        print("stream", k, "called off:", off, flush=True)
        torch.cuda.synchronize()
        called_off += off
        if off:
            time.sleep(REST)
    assert called_off > 0
    same(seq.state(), ref)


# A stream that may use half of the CUs: all workgroups at once would never be on them.
def test_stream_with_a_cu_mask_runs_group_by_group(S):
    import ctypes
    import torch
    hip = S._lib                                   # (the runtime this library runs on)
    stream = ctypes.c_void_p()
    mask = (ctypes.c_uint32 * 4)(*([0xffffffff] * 4))
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 4, mask) == 0
    seq = Sequence(S, 512, 8, 1024, 1000, 60, 2)
    assert seq.step(0)
    torch.cuda.synchronize()
    own = seq.ses.stream
    seq.ses.dec.stream = seq.ses.stream = torch.cuda.ExternalStream(stream.value)
    assert not seq.step(1)
    torch.cuda.synchronize()
    seq.ses.dec.stream = seq.ses.stream = own
    assert seq.step(1)
    assert torch.isfinite(seq.state()[0]).all()


# A wait past its limit of polls: the outputs say so, the next run reports it, and from then on the groups run one by one.
def test_wait_past_its_limit_is_reported(S):
    import torch
    seq = Sequence(S, 512, 8, 1024, 1000, 126, 2)
    for t in range(2):
        seq.step(t, variant=6)
    ref = seq.state()
    seq.ses.logits.zero_()
    torch.cuda.synchronize()
    assert seq.step(0, polls=1)
    torch.cuda.synchronize()
    assert torch.isnan(seq.ses.logits[1]).all()
    with pytest.raises(S.Sod2Error) as e:
        seq.step(0)
    assert e.value.code == -7 and "one-row step" in str(e.value)
    for t in range(2):
        assert not seq.step(t)
    same(seq.state(), ref)
