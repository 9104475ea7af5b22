"""GPU parity of the QAD distillation loss (Sec. 3.3, Eq. qad-objective) against the FP64 oracle.

Per-token KL: |kl - ref| <= 5e-5 + 1e-3 |ref| (FP32 online log-sum-exp over up to 152K terms:
the log-sum-exp values are O(10-30), a few FP32 ulps of which is ~1e-5, and the per-lane sums
carry a relative error of ~1e-5).  Gradient (bf16 output): the Q26 metric.  Top-1 agreement:
exact (comparisons of bf16 values, no arithmetic)."""
import numpy as np
import pytest

import oracle
import workloads
from tests.helpers import assert_close, bf16_to_f64, empty_bf16, from_dev, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def qf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_39223_amd as qf
    qf.lib()
    return qf


def _run(qf, zt, zs, with_grad=True, pad=0):
    L, V = zt.shape
    if pad:
        zt = np.pad(zt, ((0, 0), (0, pad)), constant_values=0x7FC0)   # NaN padding never read
        zs = np.pad(zs, ((0, 0), (0, pad)), constant_values=0x7FC0)
    t, s = to_dev(zt)[:, :V], to_dev(zs)[:, :V]
    kl = torch.empty(L, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    agree = torch.empty(L, dtype=torch.int32, device="cuda")
    grad = empty_bf16((L, V)) if with_grad else None
    qf.qad_kl(t, s, kl, loss=loss, grad=grad, agree=agree)
    torch.cuda.synchronize()
    return (from_dev(kl), float(from_dev(loss)[0]), from_dev(grad) if with_grad else None,
            from_dev(agree))


def _check(got, ref, tag=""):
    kl, loss, grad, agree = got
    rloss, rkl, rgrad, ragree = ref
    assert np.all(np.abs(kl - rkl) <= 5e-5 + 1e-3 * np.abs(rkl)), f"{tag} kl"
    assert abs(loss - rloss) <= 5e-5 + 1e-3 * abs(rloss), f"{tag} loss"
    assert np.array_equal(agree, ragree), f"{tag} agree"
    if grad is not None:
        assert_close(bf16_to_f64(grad), rgrad, f"{tag} grad")


@pytest.mark.parametrize("L,V,pad", [(37, 1000, 0), (5, 8, 0), (64, 8192, 24), (3, 151936, 0)])
def test_qad_kl_matches_oracle(qf, L, V, pad):
    d = workloads.qad_logits(L + V, L, V)
    got = _run(qf, d["zt"], d["zs"], pad=pad)
    _check(got, oracle.qad_kl(d["zt"], d["zs"]), f"L={L} V={V}")


@pytest.mark.parametrize("L,V", [
    (3, 8 * 512), (3, 8 * 512 * 8 - 8), (2, 8 * 512 * 8 + 8), (2, 8 * 512 * 12), (2, 8 * 512 * 12 + 8),
    (3, 65536), (2, 65544), (2, 8 * 1024 * 12 - 8), (2, 8 * 1024 * 13 + 8), (2, 8 * 1024 * 14),
    (1100, 520), (260, 65544)])
def test_qad_kl_kept_parts_and_row_walk(qf, L, V):
    """The ends of what a lane keeps in registers and in LDS, for both workgroup sizes, and more
    rows than workgroups; the maxima of some rows are tied with an element at the ends.

    Gradient: a probability is 2^(a - c), c = log2 of the sum (below 64: half an ulp is 2^-19,
    1.3e-6 of the probability) and the sum itself good to about 1e-6, so each is within 4e-6 of
    its own value; their difference, however small, is then rounded to bf16."""
    d = workloads.qad_logits(L + V, L, V)
    zt, zs = d["zt"].copy(), d["zs"].copy()
    for z in (zt, zs):
        top = z[np.arange(L), bf16_to_f64(z).argmax(1)]
        z[::2, V - 1 if V % 16 else V - 2] = top[::2]
        z[1::3, 0] = top[1::3]
    kl, loss, grad, agree = _run(qf, zt, zs)
    ref = oracle.qad_kl(zt, zs)
    _check((kl, loss, None, agree), ref, f"L={L} V={V}")
    p = 0.0
    for z in (bf16_to_f64(zt), bf16_to_f64(zs)):
        e = np.exp(z - z.max(1, keepdims=True))
        p = p + e / e.sum(1, keepdims=True)
    err = np.abs(bf16_to_f64(grad) - ref[2])
    assert np.all(err <= 2.0 ** -8 * np.abs(ref[2]) + 4e-6 * p / L)


def test_qad_kl_ties_and_identical_rows(qf):
    rng = np.random.default_rng(4)
    L, V = 16, 512
    zt = workloads.to_bf16(rng.integers(-3, 4, size=(L, V)).astype(np.float32))   # many ties
    zs = zt.copy()
    zs[::2] = workloads.to_bf16(rng.integers(-3, 4, size=(L // 2, V)).astype(np.float32))
    got = _run(qf, zt, zs)
    ref = oracle.qad_kl(zt, zs)
    _check(got, ref, "ties")
    assert np.all(got[0][1::2] == 0.0) or np.all(np.abs(got[0][1::2]) < 1e-6)


def test_qad_kl_loss_only_and_determinism(qf):
    d = workloads.qad_logits(7, 24, 4096)
    a = _run(qf, d["zt"], d["zs"], with_grad=True)
    b = _run(qf, d["zt"], d["zs"], with_grad=False)
    c = _run(qf, d["zt"], d["zs"], with_grad=True)
    assert np.array_equal(a[0], b[0]) and a[1] == b[1] and np.array_equal(a[3], b[3])
    assert np.array_equal(a[0], c[0]) and np.array_equal(a[2], c[2])


def test_qad_kl_no_tokens(qf):
    z = torch.empty(0, 64, dtype=torch.int16, device="cuda")
    kl = torch.empty(0, dtype=torch.float32, device="cuda")
    loss = torch.full((1,), 9.0, dtype=torch.float32, device="cuda")
    qf.qad_kl(z, z, kl, loss=loss)
    torch.cuda.synchronize()
    assert float(loss.item()) == 0.0


def test_qad_kl_full_size_sampled(qf):
    """The benchmarked shape (8192 tokens x 151936 vocabulary) in the launch configuration the
    benchmark times: per-token KL, agreement and gradient rows checked on sampled tokens
    (the oracle's per-row definition), the loss against the mean of the GPU's own per-token
    values and a sampled estimate."""
    L, V = 8192, 151936
    g = torch.Generator(device="cuda")
    g.manual_seed(0)
    t = (torch.randn(L, V, generator=g, device="cuda") * 2)
    hot = torch.randint(0, V, (L, 3), generator=g, device="cuda")
    t.scatter_add_(1, hot, torch.rand(L, 3, generator=g, device="cuda") * 8 + 6)
    s = t + torch.randn(L, V, generator=g, device="cuda") * 0.5
    zt, zs = t.to(torch.bfloat16), s.to(torch.bfloat16)
    del t, s
    kl = torch.empty(L, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    agree = torch.empty(L, dtype=torch.int32, device="cuda")
    grad = torch.empty(L, V, dtype=torch.bfloat16, device="cuda")
    qf.qad_kl(zt, zs, kl, loss=loss, grad=grad, agree=agree)
    torch.cuda.synchronize()
    rows = np.random.default_rng(1).choice(L, 12, replace=False)
    ri = torch.from_numpy(rows).cuda()
    ztr = from_dev(zt[ri].view(torch.int16))
    zsr = from_dev(zs[ri].view(torch.int16))
    _, rkl, rgrad, ragree = oracle.qad_kl(ztr, zsr)
    k = from_dev(kl)
    assert np.all(np.abs(k[rows] - rkl) <= 5e-5 + 1e-3 * np.abs(rkl))
    assert np.array_equal(from_dev(agree)[rows], ragree)
    # the oracle's gradient is for a 12-token average; the launch used 1 / 8192
    gr = bf16_to_f64(from_dev(grad[ri].view(torch.int16)))
    assert_close(gr, rgrad * 12 / L, "grad rows")
    assert abs(float(loss.item()) - k.astype(np.float64).mean()) <= 1e-6 * (1 + k.mean())


@pytest.mark.parametrize("L,V", [(256, 8 * 512 * 4), (64, 151936)])
def test_qad_kl_keeps_its_precision_where_late_chunks_dominate(qf, L, V):
    """Logits that rise along the row, so that every lane's first maximum is passed by far.  The loss
    of a row is Q / S_T + lse_S - lse_T, all below 1 here.  Its rounding: the last additions of each of
    the two merge trees (an addition's rms error is 2.5e-8 of its sum, and an addition k levels
    below the last is averaged over 2^k others: 3.5e-8), the division, logarithm and products
    (about 2e-8 each); the exponents' own (2^-22 of each) average out over the lanes.  About 8e-8
    in all; twice that is allowed (against FP64: 7e-8 measured; with log-sum-exps rounded before
    they are subtracted 4e-7, and with maxima 2^16 above the reference 5e-7)."""
    g = np.random.default_rng(L)
    t = 0.5 * g.standard_normal((L, V), dtype=np.float32) + np.linspace(-10, 0, V, dtype=np.float32)
    zt = workloads.to_bf16(t)
    zs = workloads.to_bf16(t + 0.1 * g.standard_normal((L, V), dtype=np.float32))
    kl = _run(qf, zt, zs)[0].astype(np.float64)
    ref = oracle.qad_kl(zt, zs)[1]
    assert np.sqrt(np.mean((kl - ref) ** 2)) <= 1.6e-7


@pytest.mark.parametrize("V", [8192, 151936])
def test_qad_kl_student_mask_of_the_lowest_value(qf, V):
    """A token that the student masks with the lowest bf16 value and the teacher puts above all that
    its lane has seen: the teacher-weighted gap stays finite (its exact value does)."""
    zt, zs = np.zeros((2, V), np.uint16), np.zeros((2, V), np.uint16)
    zt[:, V - 3] = workloads.to_bf16(np.array([8.0], np.float32))[0]
    zs[:, V - 3] = 0xFF7F
    kl, _, grad, agree = _run(qf, zt, zs)
    _, rkl, rgrad, ragree = oracle.qad_kl(zt, zs)
    assert np.all(np.isfinite(rkl)) and np.all(np.abs(kl / rkl - 1) <= 1e-4)
    assert np.array_equal(agree, ragree)
    assert np.all(np.abs(bf16_to_f64(grad) - rgrad) <= 2.0 ** -8 * np.abs(rgrad) + 1e-6)


@pytest.mark.parametrize("V", [8, 4096, 32776, 151936])
def test_qad_kl_of_a_distribution_with_itself(qf, V):
    """Equal logits give equal sums, so the loss and every gradient are exactly zero."""
    zt = workloads.qad_logits(V, 3, V)["zt"]
    kl, loss, grad, agree = _run(qf, zt, zt.copy())
    assert np.all(kl == 0.0) and loss == 0.0 and np.all(grad == 0) and np.all(agree == 1)


@pytest.mark.parametrize("V", [520, 12296, 32000, 65536, 65544])
def test_qad_kl_same_loss_with_and_without_gradient(qf, V):
    """The loss rows and the agreement do not depend on whether the gradient is asked for: both
    launches deal a row to as many lanes."""
    d = workloads.qad_logits(V + 1, 9, V)
    a = _run(qf, d["zt"], d["zs"], with_grad=True)
    b = _run(qf, d["zt"], d["zs"], with_grad=False)
    assert np.array_equal(a[0], b[0]) and a[1] == b[1] and np.array_equal(a[3], b[3])
    _check(b, oracle.qad_kl(d["zt"], d["zs"]), f"V={V}")
