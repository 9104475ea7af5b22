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


def test_ragged_token_count_past_the_transposed_rows(qf):
    """A ragged token count whose transposed rows are 2^22 elements and longer: the products take their
    operands in place, stored with K as their rows.  A narrow layer, dX and dW against FP64.

    dW sums 4194297 products of standard normals in FP32, about 131000 additions one after the other
    at a running size of up to 2048: a rounding of about 2e-5 of the result's rms, well inside the
    layer's tolerance."""
    M, N, K = (1 << 22) - 7, 16, 64
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    X, dY = (torch.randn(M, c, generator=g, device="cuda").to(torch.bfloat16) for c in (K, N))
    W = (torch.randn(N, K, generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    d = qf.qlinear_desc(M, N, K, "nvfp4", "none")
    Y, dX = torch.empty_like(dY), torch.empty_like(X)
    dW = torch.full((N, K), 7.0, dtype=torch.float32, device="cuda")
    ws = qf.workspace(d)
    ws.fill_(0xFF)
    qf.qlinear_fwd(d, X, W, Y, ws)
    qf.qlinear_bwd_ste(d, dY, X, W, dX, dW, ws)
    torch.cuda.synchronize()
    ref = torch.zeros(N, K, dtype=torch.float64, device="cuda")
    for i in range(0, M, 1 << 19):
        ref += dY[i:i + (1 << 19)].double().t() @ X[i:i + (1 << 19)].double()
    assert_close(from_dev(dW).astype(np.float64), from_dev(ref), "dW")
    what = oracle.fakequant(from_dev(W.view(torch.int16)), "nvfp4")
    rows = np.r_[0:300, M - 300:M]
    ri = torch.from_numpy(rows).cuda()
    got = bf16_to_f64(from_dev(dX[ri].view(torch.int16)))
    assert_close(got, oracle.linear_dx(from_dev(dY[ri].view(torch.int16)), what), "dX")


@pytest.mark.parametrize("wfmt,afmt", [("nvfp4", "none"), ("mxfp4", "mxfp4"), ("q4k", "none")])
def test_ragged_kept_workspace_after_a_forward_with_saved(qf, wfmt, afmt):
    """QF_FLAG_REUSE_WS and no saved buffer on a ragged token count, after a forward with one and after
    a forward without: the gradients of the backward from the saved buffer, bit for bit.  The
    workspace starts out as NaNs (after the former it holds no packed W)."""
    M, N, K = 1027, 136, 512
    rng = np.random.default_rng(1)
    X, W = to_dev(workloads.normal_bf16(rng, (M, K))), to_dev(workloads.normal_bf16(rng, (N, K), 0.02))
    dY = to_dev(workloads.normal_bf16(rng, (M, N)))
    outs = []
    for fwd_saved, bwd_saved in ((True, True), (True, False), (False, False)):
        d = qf.qlinear_desc(M, N, K, wfmt, afmt, flags=qf.FLAG_REUSE_WS)
        sv, ws = qf.saved_buffer(d), qf.workspace(d)
        ws.fill_(0xFF)
        Y, dX = empty_bf16((M, N)), empty_bf16((M, K))
        dW = torch.full((N, K), 7.0, dtype=torch.float32, device="cuda")
        qf.qlinear_fwd(d, X, W, Y, ws, saved=sv if fwd_saved else None)
        qf.qlinear_bwd_ste(d, dY, X, W, dX, dW, ws, saved=sv if bwd_saved else None)
        torch.cuda.synchronize()
        outs.append((dX, dW))
    for dX, dW in outs[1:]:
        assert torch.equal(dX, outs[0][0]) and torch.equal(dW, outs[0][1])
