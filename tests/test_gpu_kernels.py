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


# fp32 contractions: 16 x 16 tiles with k split over 8 waves (rows and columns of one tile and one more, k shorter than
# one chunk per wave, k not a multiple of 4, k longer than one round of loads), 32 x 32 tiles, 64 x 64 FMA tiles
@pytest.mark.parametrize("M,N,K,trans_b,batch", [
    (2, 64, 768, 1, 1), (8, 1, 64, 1, 1), (16, 16, 16, 1, 1), (17, 15, 77, 0, 3), (77, 77, 64, 1, 4), (77, 64, 77, 0, 4),
    (33, 47, 1030, 1, 1), (128, 1024, 256, 1, 1), (513, 545, 260, 1, 1), (300, 300, 131, 0, 4), (1473, 1409, 40, 1, 1)])
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
