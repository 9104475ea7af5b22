"""The layer's backward on token counts that are not multiples of 8: the transposed operands are
padded with zeros to whole 16-byte groups, dY^T by the dX launch (both large tiles) or the transpose
kernel, A_hat^T by the transpose, the transposing quantizer or the transposing dequantizer.  dX and
dW against FP64 products, and dW bit-identical whichever kernel wrote dY^T; the workspace starts
out as NaNs, so that nothing past the last token may be read from it."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import assert_close, bf16_to_f64, empty_bf16, from_dev, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def qf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_39223_amd as qf
    qf.lib()
    return qf


@pytest.mark.parametrize("M,N,K,wfmt,afmt,saved", [
    (1, 72, 64, "nvfp4", "none", True), (13, 264, 256, "q4k", "none", True),
    (63, 40, 544, "mxfp4", "mxfp4", False), (65, 40, 512, "nvfp4", "nvfp4", True),
    (2043, 136, 4096, "nvfp4", "none", True),       # dX in 256 x 128 tiles, writing dY^T
    (2046, 136, 1920, "mxfp4", "mxfp4", True),      # 15 tile columns
    (4099, 72, 4096, "mxfp4", "mxfp4", True),       # dX in 256 x 256 tiles, writing dY^T
    (4097, 72, 4096, "nvfp4", "none", False)])
def test_ragged_token_counts(qf, M, N, K, wfmt, afmt, saved):
    rng = np.random.default_rng(M + N + K)
    Xh, Wh = workloads.normal_bf16(rng, (M, K)), workloads.normal_bf16(rng, (N, K), 0.02)
    dYh = workloads.normal_bf16(rng, (M, N))
    X, W, dY = to_dev(Xh), to_dev(Wh), to_dev(dYh)
    g = float(oracle.amax(Xh)) if afmt == "nvfp4" else None
    a_amax = torch.tensor([g], device="cuda") if g is not None else None
    d = qf.qlinear_desc(M, N, K, wfmt, afmt, a_amax=a_amax)
    sv = qf.saved_buffer(d) if saved else None
    outs = []
    for want_dx in (True, False):
        ws = qf.workspace(d)
        ws.fill_(0xFF)
        Y, dX = empty_bf16((M, N)), empty_bf16((M, K)) if want_dx else None
        dW = torch.full((N, K), 7.0, dtype=torch.float32, device="cuda")
        qf.qlinear_fwd(d, X, W, Y, ws, saved=sv)
        qf.qlinear_bwd_ste(d, dY, X, W, dX, dW, ws, saved=sv)
        torch.cuda.synchronize()
        outs.append((dX, from_dev(dW)))
    assert np.array_equal(outs[0][1].view(np.uint32), outs[1][1].view(np.uint32))
    what = oracle.fakequant(Wh, wfmt)
    ahat = oracle.fakequant(Xh, afmt, g) if afmt != "none" else Xh
    assert_close(outs[0][1].astype(np.float64), oracle.linear_dw(dYh, ahat), "dW")
    assert_close(bf16_to_f64(from_dev(outs[0][0])), oracle.linear_dx(dYh, what), "dX")
