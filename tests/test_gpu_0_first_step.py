"""The first decode step of the process.  (First of the GPU tests, so that it is one.)"""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_first_step_while_another_thread_captures(S_lib):
    """What the one-kernel step sets up once (pinned memory, an event) is set up while another thread captures a stream in
    the mode that forbids every thread such calls: the step runs, the capture holds."""
    import torch
    from paper_2403_00176_amd.session import DecoderSession
    from workloads import configs
    w = configs.decoder(layers=2, hidden=256, heads=4, ffn=512, vocab=200, p_range=(1, 512), t_max=4, n_prompts=1)
    ses = DecoderSession(w.prefill, w.decode, w.t_max)
    ses.upload_weights(w.make_weights_by_name())
    ses.start(20, 200)
    ses.prefill(torch.arange(20).to(ses.device))
    x = torch.zeros(1000, device=ses.device)
    torch.cuda.synchronize()
    result = []

    def step():
        try:
            torch.cuda.set_device(ses.device)
            result.append({e["kernel"] for e in S_lib.sod2_run_trace(ses.decode(0))})
        except Exception as e:                     # noqa: BLE001 (shown by the assertion below)
            result.append(e)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="global"):
        x += 1
        thread = threading.Thread(target=step)
        thread.start()
        thread.join()
        x += 1
    torch.cuda.synchronize()
    assert result == [{23}], result
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert (x == 2 * (k + 1)).all()
    assert torch.isfinite(ses.logits[1].float()).all() and ses.logits[1].float().abs().max() > 0
