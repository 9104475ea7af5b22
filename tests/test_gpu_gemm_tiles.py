"""The dense GEMM's tiles: one shape per tile of the choice (the smallest ceil(tiles / 256) (rows +
columns) on the 256-unit device), each ragged in both directions, over contraction depths below
one stage, at whole stage groups, with a partial last group and a partial last stage; contractions
long enough for the L2 prefetch; the FP32 split of the last round; and the forms that must agree
bit for bit (A^T written along, weight decoded inside) at shapes that run in the large tiles.
Expected values are FP64 products, tolerance the layer's (bf16 rounding of the result)."""
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


def _operands(M, N, K):
    rng = np.random.default_rng(M * 3 + N * 5 + K)
    return workloads.normal_bf16(rng, (M, K)), workloads.normal_bf16(rng, (N, K))


def _check(qf, M, N, K, c32, ws=None):
    A, B = _operands(M, N, K)
    C = torch.full((M, N), 7, dtype=torch.float32 if c32 else torch.int16, device="cuda")
    qf.gemm_bf16(M, N, K, to_dev(A), K, 1, to_dev(B), K, 1, C, N, c32, ws=ws)
    torch.cuda.synchronize()
    got = from_dev(C)
    # every column of up to 96 rows: the first and last tile rows and some between
    rows = np.unique(np.concatenate([np.arange(min(M, 32)), np.arange(max(0, M - 32), M),
                                     np.linspace(0, M - 1, 32).astype(int)]))
    g = got[rows].astype(np.float64) if c32 else bf16_to_f64(got[rows])
    assert_close(g, oracle.linear_fwd(np.ascontiguousarray(A[rows]), B), f"{M}x{N}x{K} c32={c32}")


TILES = [(9, 4088), (60, 4088), (248, 4088), (504, 4088), (1016, 4088), (2040, 4080), (4104, 4104)]


@pytest.mark.parametrize("c32", [0, 1])
@pytest.mark.parametrize("M,N", TILES, ids=["16x16", "32x32", "64x64", "128x64", "128x128",
                                            "256x128", "256x256"])
def test_every_tile_at_its_edges(qf, M, N, c32):
    for K in (40, 64, 200, 576, 1096):
        _check(qf, M, N, K, c32)


@pytest.mark.parametrize("M,N,K,c32", [(2040, 4080, 6200, 0), (4104, 4104, 6152, 1),
                                       (4104, 4104, 6144, 0)])
def test_long_contractions_prefetch(qf, M, N, K, c32):
    _check(qf, M, N, K, c32)


def test_split_of_the_last_round(qf):
    # 8 x 33 tiles: one full round and 8 tiles that run as two K halves each
    M, N, K = 2048, 8448, 200
    _check(qf, M, N, K, 1, ws=qf.gemm_workspace(M, N, 1))


@pytest.mark.parametrize("M,N,K", [(4096, 1920, 200), (8200, 3840, 136), (4104, 4104, 200),
                                   (2048, 4096, 6208)],
                         ids=["256x128 two pieces", "256x256 two pieces", "256x256 one piece",
                              "256x128 prefetch"])
def test_transposed_a_output_in_large_tiles(qf, M, N, K):
    A, B = _operands(M, N, K)
    Ad, Bd = to_dev(A), to_dev(B)
    at = torch.full((K, M + 12), 0x1234, dtype=torch.int16, device="cuda")
    C, C2 = empty_bf16((M, N)), empty_bf16((M, N))
    qf.gemm_bf16_at(M, N, K, Ad, K, Bd, K, C, N, at, M + 12)
    qf.gemm_bf16(M, N, K, Ad, K, 1, Bd, K, 1, C2, N, 0)
    torch.cuda.synchronize()
    assert torch.equal(C, C2)
    a_t = from_dev(at).view(np.uint16)
    assert np.array_equal(a_t[:, :M], A.T) and np.all(a_t[:, M:] == 0x1234)


@pytest.mark.parametrize("wfmt", ["nvfp4", "mxfp4", "q4k"])
def test_decoded_weight_equals_materialized_in_256x256_tiles(qf, wfmt):
    M, N, K = 4104, 4104, 1024
    X, W = _operands(M, N, K)
    Ys = []
    for flags in (qf.FLAG_DECODE_IN_GEMM, 0):
        d = qf.qlinear_desc(M, N, K, wfmt, "none", flags=flags)
        Y = empty_bf16((M, N))
        qf.qlinear_fwd(d, to_dev(X), to_dev(W), Y, qf.workspace(d))
        Ys.append(Y)
    torch.cuda.synchronize()
    assert torch.equal(Ys[0], Ys[1])


@pytest.mark.parametrize("c32", [0, 1])
def test_fragment_order_equals_row_order_in_256x256_tiles(qf, c32):
    M, N, K = 4104, 4104, 1024
    A, B = _operands(M, N, K)
    Ad, Bd = to_dev(A), to_dev(B)
    Bf = torch.empty(qf.fragment_bytes(N, K) // 2, dtype=torch.int16, device="cuda")
    qf.pack_fragments(Bd, Bf)
    dt = torch.float32 if c32 else torch.int16
    C1, C2 = (torch.full((M, N), v, dtype=dt, device="cuda") for v in (3, 5))
    qf.gemm_bf16_fragb(M, N, K, Ad, K, Bf, C1, N, c32)
    qf.gemm_bf16(M, N, K, Ad, K, 1, Bd, K, 1, C2, N, c32)
    torch.cuda.synchronize()
    assert torch.equal(C1, C2)


@pytest.mark.parametrize("M,N,K", [(2048, 2048, 1024), (2040, 2048, 1088), (1024, 2048, 1024),
                                   (1024, 2044, 1088), (2048, 2048, 200), (1016, 2040, 136)],
                         ids=["128x128", "128x128 odd stages", "128x64", "128x64 odd stages",
                              "128x128 tail", "128x64 tail"])
def test_k_halves_in_small_tiles(qf, M, N, K):
    """FP32 with a workspace, in the small kernel's two largest tiles: the sum of the two K halves that
    the large tiles form, so bit-identical to the fragment-order product, which runs in those."""
    ws = qf.gemm_workspace(M, N, 1)
    assert ws is not None
    _check(qf, M, N, K, 1, ws=ws)
    if K % 64:
        return
    A, B = _operands(M, N, K)
    Ad, Bd = to_dev(A), to_dev(B)
    Bf = torch.empty(qf.fragment_bytes(N, K) // 2, dtype=torch.int16, device="cuda")
    qf.pack_fragments(Bd, Bf)
    C1, C2 = (torch.full((M, N), v, dtype=torch.float32, device="cuda") for v in (3, 5))
    qf.gemm_bf16_fragb(M, N, K, Ad, K, Bf, C1, N, 1, ws=ws)
    qf.gemm_bf16(M, N, K, Ad, K, 1, Bd, K, 1, C2, N, 1, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(C1, C2)
