"""Wide workgroups with split float32 operands (three bf16 pieces), one and two row blocks, two groups of two row blocks, and the
one-wave tiles whose K is split over waves next to a pass at x of few chunks: every score against the oracle."""
import numpy as np
import pytest
import torch

from paper_1805_10032_amd import workloads as WL
from tests._util import SCORE_TOL, npy, oracle_terms, rows_to_gpu, score_error

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1805_10032_amd import binding
    binding.load_library()
    return binding


def _run(B, w, row_align, G=None):
    dev = torch.device("cuda", 0)
    mdl = B.ZenoModel(w.dims, w.has_bias, w.loss, w.fwd)
    G = rows_to_gpu(B, w.G if G is None else G, row_align, dev)
    B.profile_enable(True)
    try:
        s = B.zeno_score(mdl, w.x.to(dev), G, w.features.to(dev), w.gamma, w.rho, labels=w.labels.to(dev))
        torch.cuda.synchronize()
        recs = [r for r in B.profile_collect(detail=True) if r["kernel"] == "layer_cand"]
    finally:
        B.profile_enable(False)
    return npy(s), recs


def _workload(name, dims, m, n_r, fwd="fp32", bias=True):
    return WL.make_mlp_workload(name, 300 + n_r, dims, m, m // 3, n_r, 0.05, 1e-3, fwd, seed=m, has_bias=bias, n_flip=m // 6,
                                n_noise=m // 6, noise_std=2.0, worker_batch=16)


@pytest.mark.parametrize("n_r", [1, 32, 33, 64, 65, 97, 128])
@pytest.mark.parametrize("dims,m,row_align,bias", [
    ([512, 1024, 512, 10], 64, 32, True),     # four and eight waves, line-aligned rows
    ([200, 1030, 500, 10], 57, 1, True),      # ragged K, tiles beyond the matrix, packed rows
    ([130, 520, 260], 100, 4, False),         # three chunks: no steady loop
])
def test_split_operands(B, dims, m, row_align, bias, n_r):
    """Both sides of every number of row blocks: 33 samples are two blocks, 65 two groups of two."""
    w = _workload("split", dims, m, n_r, bias=bias)
    s, recs = _run(B, w, row_align)
    wide = [r for r in recs if r["waves"] >= 4]
    assert len(wide) >= 2 and all(r["row_blocks"] == (1 if n_r <= 32 else 2 if n_r <= 64 else 4) for r in wide), recs
    err = score_error(s, *oracle_terms(w))
    assert np.all(err <= SCORE_TOL["fp32"]), (float(err.max()), int(err.argmax()))


@pytest.mark.parametrize("n_r", [32, 48, 100])
@pytest.mark.parametrize("row_align", [1, 32])
def test_a_product_keeps_24_bits(B, n_r, row_align):
    """Sums of one product, so that nothing averages out: one weight of the first layer moves one hidden unit, and one weight of x
    carries it through the second.  In units of 2^-24: at most 1 for what the six piece products leave out and 1 for the rounding
    of the sum, at each of the two layers, and 1 for the score; everything else is exact.  Factors close to 1 + 2^-7 from below have a
    middle piece of 2^-16 and hardly a last one, so that nothing is left out (leading pieces cut toward zero would leave most behind
    there, 2.8 to 4.7 units in all)."""
    K, N, N2 = 512, 1024, 512
    w = _workload("bits", [K, N, N2, 10], 64, n_r)
    w.dims, w.loss, w.has_bias, w.gamma, w.rho = [K, N, N2, 1], "squared", True, 2.0 ** -4, 0.0
    w.labels, w.targets = None, torch.full((n_r,), -1024.0)
    b0, w1 = N * K, N * K + N
    b1 = w1 + N2 * N
    w2 = b1 + N2
    d = w2 + N2 + 1
    unit, row, col = 37, 11, 70
    w.x, w.G = torch.zeros(d), torch.zeros((64, d))
    near = 1 + 2.0 ** -7 - 2.0 ** -15 + 2.0 ** -16 - torch.arange(1, 65, dtype=torch.float64) * 2.0 ** -23
    gen = torch.Generator().manual_seed(3)
    u = torch.where(torch.arange(64) < 40, near, 1 + torch.rand(64, generator=gen, dtype=torch.float64)).float()
    w.features = torch.zeros((n_r, K))
    w.features[:, col] = near[9]
    w.G[:, unit * K + col] = -u
    w.x[b0 + unit], w.x[w1 + row * N + unit], w.x[w2 + row] = 1.0, near[21], 1.0
    dev = torch.device("cuda", 0)
    mdl = B.ZenoModel(w.dims, w.has_bias, w.loss, w.fwd)
    s = npy(B.zeno_score(mdl, w.x.to(dev), rows_to_gpu(B, w.G, row_align, dev), w.features.to(dev), w.gamma, w.rho, targets=w.targets.to(dev)))
    ref = oracle_terms(w)[0]
    err = np.abs(s - ref) / np.abs(ref) * 2.0 ** 24
    assert err[:40].max() <= 3.1 and err[40:].max() <= 5.1, (float(err[:40].max()), float(err[40:].max()))


def test_values_that_are_not_finite(B):
    """Infinities, NaNs of any payload and the largest floats in a few candidates: their scores are not finite, and nobody else's
    changes.  A NaN with its payload in the lower half must not become infinity on the way."""
    w = _workload("special", [512, 1024, 512, 10], 64, 32)
    clean, _ = _run(B, w, 32)
    G = w.G.clone()
    col = 3 * 512 + 7   # inside the first layer's weights
    second = 1024 * 512 + 1024 + 5 * 1024 + 11
    bits = torch.tensor([0x7f800001, -8388607], dtype=torch.int32).view(torch.float32)   # NaNs, payload in the lower half
    G[0, col], G[1, col], G[2, col], G[3, col] = float("inf"), float("-inf"), float("nan"), 3.402e38
    G[4].view(-1)[col:col + 1] = bits[:1]
    G[5].view(-1)[second:second + 1] = bits[1:]
    G[6, second], G[7, second] = float("inf"), -3.402e38
    s, recs = _run(B, w, 32, G)
    assert all(r["waves"] >= 4 for r in recs[:2]), recs
    assert not np.isfinite(s[[0, 1, 2, 4, 5, 6]]).any(), s[:8]
    assert np.isnan(s[[2, 4, 5]]).all(), s[:8]
    assert (np.isnan(s[[3, 7]]) | (s[[3, 7]] < -1e30)).all(), s[:8]
    assert np.array_equal(s[8:], clean[8:])


NAN_BITS = {1.0: 0x7f800001, -1.0: -8388607}   # NaNs that are infinity, of either sign, without their lower half


def _nan(sign):
    return torch.tensor([NAN_BITS[sign]], dtype=torch.int32).view(torch.float32)


def _all_scores_nan(B, w, place, sign):
    """place(w, v) puts v where the test wants the NaN.  An infinity of the same sign there must leave every score finite (so
    that a NaN taken for one would be seen), the NaN itself no score at all."""
    place(w, torch.tensor([sign * float("inf")]))
    with np.errstate(invalid="ignore"):
        assert np.isfinite(oracle_terms(w)[0]).all()
    place(w, _nan(sign))
    s, recs = _run(B, w, 32)
    assert any(r["waves"] >= 4 for r in recs), recs
    assert np.isnan(s).all(), s


@pytest.mark.parametrize("dims,n_r", [([512, 1024, 512, 10], 32), ([512, 1024, 512, 10], 40), ([512, 1024, 512, 10], 100),
                                      ([1088, 1024, 512, 10], 9)])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_a_nan_in_the_batch(B, dims, n_r, sign):
    """One feature of one sample, packed by the first launch (up to 1024 inputs and 32 samples) or by a launch of its own.  As an
    infinity it would push the sample's hidden features to minus infinity, at x and at the candidates, and from there to zero."""
    w = _workload("nanbatch", dims, 64, n_r)
    col, K, N = 70, dims[0], dims[1]
    w.x[:N * K].view(N, K)[:, col] = -0.01 * sign
    w.G[:, :N * K].view(-1, N, K)[:, :, col] = 0.01 * sign

    def place(w, v):
        w.features[min(3, n_r - 1), col:col + 1] = v
    _all_scores_nan(B, w, place, sign)


@pytest.mark.parametrize("n_r", [32, 48, 100])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_a_nan_in_x_of_a_wide_output_layer(B, n_r, sign):
    """The pass at x rides in the candidates' launch, on split operands.  As an infinity it would take one class's logit to minus
    infinity for every sample, and no sample has that label."""
    w = _workload("nanx1", [512, 1024], 64, n_r)
    col, cls = 70, 33
    w.features[:, col] = -sign * w.features[:, col].abs().clamp_min(0.1)
    w.G[:, cls * 512 + col] = 0.0
    w.labels[w.labels == cls] = cls + 1

    def place(w, v):
        w.x[cls * 512 + col:cls * 512 + col + 1] = v
    _all_scores_nan(B, w, place, sign)


@pytest.mark.parametrize("n_r", [32, 48, 100])
def test_a_nan_in_x_of_a_wide_hidden_layer(B, n_r):
    """A weight of the second hidden layer: the pass at x writes it in operand order, where every candidate's second product reads it.
    As minus infinity it would take one hidden feature, whose input is positive for all samples, to zero."""
    dims = [512, 1024, 512, 10]
    w = _workload("nanx2", dims, 64, n_r)
    unit, row, b0, w1 = 5, 11, 512 * 1024, 512 * 1024 + 1024
    w.x[b0 + unit], w.G[:, b0 + unit] = 100.0, -1.0                       # positive at x, larger at every candidate
    w.G[:, unit * 512:(unit + 1) * 512] = 0.0
    at = w1 + row * 1024 + unit
    w.G[:, at] = 0.0

    def place(w, v):
        w.x[at:at + 1] = v
    _all_scores_nan(B, w, place, -1.0)


@pytest.mark.parametrize("n_r", [32, 48, 100])
@pytest.mark.parametrize("row_align", [1, 32])
def test_operands_near_the_end_of_the_range(B, n_r, row_align):
    """Finite operands from 3.396e38 on, which a leading piece rounded to nearest takes to infinity, in the batch, in x's first
    layer and in x's second layer, next to factors of 1e-31 and less: every score is finite and right.  (A candidate's own values of
    that size make its squared norm infinite.)"""
    dims = [512, 1024, 512, 10]
    w = _workload("top", dims, 64, n_r)
    top, gen = 3.4e38, torch.Generator().manual_seed(n_r)

    def noise(*shape, std):
        return torch.randn(shape, generator=gen) * std
    K, N, b0, w1 = 512, 1024, 512 * 1024, 512 * 1024 + 1024
    b1 = w1 + 512 * 1024
    x0, G0 = w.x[:N * K].view(N, K), w.G[:, :N * K].view(64, N, K)
    x1, G1 = w.x[w1:b1].view(512, N), w.G[:, w1:b1].view(64, 512, N)
    x2, G2 = w.x[b1 + 512:b1 + 512 + 5120].view(10, 512), w.G[:, b1 + 512:b1 + 512 + 5120].view(64, 10, 512)
    w.features[:, 70] = top * torch.where(torch.rand(n_r, generator=gen) < 0.5, 1.0, -1.0)     # in the batch: z about 3e7
    x0[:, 70], G0[:, :, 70] = noise(N, std=1e-31), noise(64, N, std=1e-32)
    x0[:, 71], w.features[:, 71], G0[:, :, 71] = top, noise(n_r, std=1e-31), 0.0               # in x
    x1 *= 1e-7
    G1 *= 1e-7
    unit = 5                                                                                   # in x's second layer
    x0[unit], G0[:, unit], w.x[b0 + unit], w.G[:, b0 + unit] = 0.0, 0.0, 1e-31, noise(64, std=1e-32)
    x1[11, unit], G1[:, 11, unit] = -top, 0.0
    x1[12, unit], G1[:, 12, unit] = top, 0.0
    x2[:, 12] *= 1e-7
    G2[:, :, 12] *= 1e-7
    s, recs = _run(B, w, row_align)
    assert all(r["waves"] >= 4 for r in recs[:2]), recs
    s_ref, scale = oracle_terms(w)
    assert np.isfinite(s_ref).all()
    err = score_error(s, s_ref, scale)
    assert np.all(err <= SCORE_TOL["fp32"]), (float(err.max()), int(err.argmax()))


@pytest.mark.parametrize("row_align", [1, 32])
@pytest.mark.parametrize("dims,m,slices", [
    ([512, 1000], 24, 1), ([512, 1000], 25, 1), ([512, 1000], 31, 1),   # 200, 208 and 256 workgroups
    ([500, 1000], 32, 1),                                               # 264; ragged K
    ([768, 1201], 7, 3), ([1114, 1278], 8, 2),                          # slices: 240 and 180
])
def test_both_kinds_of_products(B, dims, m, slices, row_align):
    """Both sides of the line between float32 matrix instructions and split operands: packed rows take the former in launches of 205 to
    256 workgroups."""
    w = _workload("kinds", dims, m, 9)
    s, (rec,) = _run(B, w, row_align)
    assert (rec["waves"], rec["k_slices"]) == (4, slices), rec
    err = score_error(s, *oracle_terms(w))
    assert np.all(err <= SCORE_TOL["fp32"]), (float(err.max()), int(err.argmax()))


@pytest.mark.parametrize("n_r", [32, 48, 100])
def test_candidates_with_the_largest_floats(B, n_r):
    """Weights of 3.402e38, which the split rounds to infinity, whose inputs are zero or not: the squared norm is infinite, the candidate
    ranks last, and nobody else's score changes.  Without them the same rows score as the oracle says, next to weights of 1e19 (the
    largest whose squares do not overflow) whose inputs are zero."""
    dims = [512, 1024, 512, 10]
    w = _workload("topzero", dims, 64, n_r)
    cols = torch.tensor([5, 300])   # in the first tile, and in one that the steady loop takes
    w.features[:, cols] = 0.0
    b0, w1 = 512 * 1024, 512 * 1024 + 1024
    G0, G1 = w.G[:, :b0].view(64, 1024, 512), w.G[:, w1:w1 + 512 * 1024].view(64, 512, 1024)
    G0[4][7, cols] = 1e19
    clean, recs = _run(B, w, 32)
    assert all(r["waves"] >= 4 for r in recs[:2]), recs
    assert np.all(score_error(clean, *oracle_terms(w)) <= SCORE_TOL["fp32"])
    G0[0][7, cols], G0[1][1023, 17], G1[2][100, 21], G0[3][7, cols] = 3.402e38, -3.402e38, 3.402e38, float("inf")
    s, _ = _run(B, w, 32)
    assert np.all(np.isnan(s[:4]) | (s[:4] == -np.inf)), s[:4]
    assert np.array_equal(s[4:], clean[4:])
    G = w.G.to("cuda")
    _, selected = B.zeno_aggregate(G, torch.from_numpy(s).to("cuda"), 4)
    assert selected.tolist() == list(range(4, 64))


@pytest.mark.parametrize("dims,m,n_r,fwd,row_align", [
    ([784, 256, 128, 10], 20, 32, "fp32", 1),    # the pass at x has four and two chunks next to 13 and four
    ([512, 30, 200], 20, 20, "fp32", 32),        # ... one chunk: three of four waves have none
    ([1000, 100, 40, 7], 24, 40, "bf16", 1),
    ([300, 64, 64, 2], 9, 100, "bf16", 4),       # two waves a tile, one chunk each
    ([256, 100, 64, 10], 40, 70, "fp32", 1),
])
def test_k_split_next_to_a_short_pass_at_x(B, dims, m, n_r, fwd, row_align):
    w = _workload("shortk", dims, m, n_r, fwd)
    s, recs = _run(B, w, row_align)
    assert any(r["waves"] == 1 and r["k_split"] > 1 and r["merged"] for r in recs), recs
    err = score_error(s, *oracle_terms(w))
    assert np.all(err <= SCORE_TOL[fwd]), (float(err.max()), int(err.argmax()))
