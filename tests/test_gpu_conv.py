"""GPU parity of zeno_score with a convolutional f_r (Section 6.1's model class on synthetic shapes)
against the float64 CPU oracle, through the C ABI: every candidate's score at the fp32 tolerance,
the selection against the oracle's scores, the aggregate."""
import numpy as np
import pytest
import torch

from oracle import zeno_oracle as O
from paper_1805_10032_amd import workloads as WL
from tests._util import AGG_TOL, SCORE_TOL, check_selection, npy, score_error

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1805_10032_amd import binding
    binding.load_library()
    return binding


def _gpu_scores(B, w, static=False):
    dev = torch.device("cuda", 0)
    mdl = B.ZenoCnnModel(w.desc, w.loss)
    assert mdl.num_params == w.d == O.cnn_num_params(w.desc)
    lab = None if w.labels is None else w.labels.to(dev)
    tgt = None if w.targets is None else w.targets.to(dev)
    fn = B.zeno_score_static if static else B.zeno_score
    s = fn(mdl, w.x.to(dev), w.G.contiguous().to(dev), w.features.to(dev), w.gamma, w.rho, labels=lab, targets=tgt)
    torch.cuda.synchronize()
    return s


def _check(B, w, tol=SCORE_TOL["fp32"]):
    s_gpu = _gpu_scores(B, w)
    s_ref, scale = O.cnn_scores(npy(w.x), npy(w.G), w.gamma, w.rho, w.desc, w.loss, npy(w.features), npy(w.labels),
                                npy(w.targets))
    err = score_error(npy(s_gpu), s_ref, scale)
    assert np.all(err <= tol), (w.name, float(np.nanmax(err)), int(np.nanargmax(err)))
    G = w.G.contiguous().cuda()
    out, sel = B.zeno_aggregate(G, s_gpu, w.b)
    torch.cuda.synchronize()
    check_selection(npy(sel), s_ref, w.b, tol, scale)
    ref, _ = O.zeno_aggregate(npy(w.G), npy(s_gpu), w.b)
    assert np.linalg.norm(npy(out).astype(np.float64) - ref) <= AGG_TOL * np.linalg.norm(ref)
    return err


CASES = [
    # desc, m, b, n_r
    (dict(in_h=6, in_w=5, in_c=2, conv_c=[4, 3], conv_stride=[1, 2], fc_out=3, has_bias=True), 5, 1, 6),
    (dict(in_h=8, in_w=8, in_c=3, conv_c=[8, 8, 16, 16], conv_stride=[1, 2, 1, 2], fc_out=10, has_bias=True), 9, 3, 4),
    (dict(in_h=7, in_w=9, in_c=1, conv_c=[33], conv_stride=[1], fc_out=5, has_bias=False), 4, 1, 3),          # one convolution, 33 channels
    (dict(in_h=5, in_w=5, in_c=3, conv_c=[5, 7, 9], conv_stride=[2, 1, 2], fc_out=4, has_bias=True), 6, 2, 1),   # one sample, odd widths
    (dict(in_h=12, in_w=12, in_c=3, conv_c=[16, 40], conv_stride=[1, 1], fc_out=10, has_bias=True), 8, 2, 33),  # two sample blocks, two channel tiles
    (dict(in_h=4, in_w=4, in_c=8, conv_c=[8], conv_stride=[1], fc_out=1, has_bias=True), 5, 1, 7),              # squared loss
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_cnn_small_shapes(B, case):
    desc, m, b, n_r = CASES[case]
    loss = "squared" if desc["fc_out"] == 1 else "softmax_ce"
    q = min(2, m - 1)
    w = WL.make_cnn_workload(f"cnn{case}", 30 + case, desc, m, b, n_r, 0.1, 1e-3, seed=case, loss=loss,
                             n_flip=min(1, q), n_noise=q - min(1, q), noise_std=0.5)
    _check(B, w)


def test_cnn_paper_shaped(B):
    """The shape of the paper's experiments (Section 6: 32 x 32 x 3 images, four convolutions and one fully
    connected layer, 10 classes, m = 20 workers of which q = 8 fail, n_r = 4, gamma = 0.1, rho = 5e-4); the
    widths 32-32-64-64 and the strides are this test's choice.  Sign-flipped rows (-4 x the honest mean)."""
    desc = dict(in_h=32, in_w=32, in_c=3, conv_c=[32, 32, 64, 64], conv_stride=[1, 2, 1, 2], fc_out=10, has_bias=True)
    w = WL.make_cnn_workload("cnn_paper", 37, desc, 20, 8, 4, 0.1, 5e-4, n_flip=8, worker_batch=16)
    _check(B, w)


def test_cnn_on_the_static_scratch_array(B):
    """zeno_score_static serves convolutional models as well (same kernels, bit for bit) while their scratch fits."""
    desc, m, b, n_r = CASES[1]
    w = WL.make_cnn_workload("cnn_static", 39, desc, m, b, n_r, 0.1, 1e-3, n_flip=1)
    assert torch.equal(_gpu_scores(B, w, static=True), _gpu_scores(B, w))


@pytest.mark.parametrize("hw,conv_c,m,n_r", [
    (14, [32, 32, 64, 64], 20, 4),    # kernel fragments and split maps fit the array
    (16, [32, 32, 64, 64], 20, 4),    # they do not, the plain maps do
    (32, [32, 32, 64, 64], 10, 4),
    (8, [64, 48], 23, 2),
])
def test_cnn_static_scratch_and_workspace_sum_in_the_same_order(B, hw, conv_c, m, n_r):
    """Bit for bit the same scores from both entry points for every model that the static array holds."""
    desc = dict(in_h=hw, in_w=hw, in_c=3, conv_c=conv_c, conv_stride=[1, 2, 1, 2][:len(conv_c)], fc_out=10, has_bias=True)
    w = WL.make_cnn_workload("cnn_static", 40, desc, m, 3, n_r, 0.1, 1e-3, n_flip=2, worker_batch=4)
    _check(B, w)
    assert torch.equal(_gpu_scores(B, w, static=True), _gpu_scores(B, w))


def test_cnn_beyond_the_static_scratch_array(B):
    desc = dict(in_h=32, in_w=32, in_c=3, conv_c=[32, 32, 64, 64], conv_stride=[1, 2, 1, 2], fc_out=10, has_bias=True)
    w = WL.make_cnn_workload("cnn_static", 41, desc, 20, 3, 4, 0.1, 1e-3, worker_batch=2)
    with pytest.raises(B.ZenoError) as e:
        _gpu_scores(B, w, static=True)
    assert e.value.status == 2


def test_cnn_nonfinite_rows_and_workspace_contents(B):
    desc = dict(in_h=6, in_w=6, in_c=2, conv_c=[6, 6], conv_stride=[1, 2], fc_out=3, has_bias=True)
    w = WL.make_cnn_workload("cnn_nf", 38, desc, 7, 2, 5, 0.1, 1e-3)
    w.G[1, 3] = float("nan")            # a kernel entry of the first convolution
    w.G[4, -1] = float("inf")           # the last bias of the fully connected layer
    dev = torch.device("cuda", 0)
    mdl = B.ZenoCnnModel(w.desc, w.loss)
    args = (mdl, w.x.to(dev), w.G.contiguous().to(dev), w.features.to(dev), w.gamma, w.rho)
    out = []
    for fill in (0.0, float("nan")):    # the scratch memory is written before it is read
        ws = B.alloc_workspace(mdl, w.m, w.n_r, dev)
        ws.view(torch.float32).fill_(fill)
        out.append(npy(B.zeno_score(*args, labels=w.labels.to(dev), workspace=ws)))
    assert np.array_equal(out[0], out[1], equal_nan=True)
    s = out[0].astype(np.float64)
    for i in (1, 4):
        assert np.isnan(s[i]) or s[i] == -np.inf
    ok = [i for i in range(w.m) if i not in (1, 4)]
    s_ref, scale = O.cnn_scores(npy(w.x), npy(w.G), w.gamma, w.rho, w.desc, w.loss, npy(w.features), npy(w.labels), rows=ok)
    assert np.all(score_error(s[ok], s_ref, scale) <= SCORE_TOL["fp32"])


FRAGMENTS = [
    # (in_h, in_w, in_c, channels, strides), m, n_r
    ((32, 32, 3, [32, 32, 64, 64], [1, 2, 1, 2]), 7, 3),   # whole rows per tile; two channel tiles
    ((9, 7, 1, [24, 40, 33], [1, 2, 1]), 5, 4),            # units of one group of eight channels; tiles across samples; a tile of one channel
    ((5, 5, 8, [16, 16], [2, 2]), 3, 1),                   # eight channels of features; fewer positions than a tile
    ((12, 10, 2, [48, 16, 96, 16], [1, 1, 2, 1]), 4, 9),   # three units, three channel tiles
    ((33, 31, 3, [64], [2]), 3, 2),                        # one convolution: straight into the fully connected layer
]


@pytest.mark.parametrize("case", range(len(FRAGMENTS)))
def test_cnn_fragments_and_split_maps(B, case):
    """Models that take reordered kernels and maps: against the oracle, with whatever the workspace held before, and with a
    workspace that lacks room for them (float32 sums in another order: 4 eps per addition of some 600 on 4 layers at most)."""
    (h, w_, c, conv_c, conv_stride), m, n_r = FRAGMENTS[case]
    desc = dict(in_h=h, in_w=w_, in_c=c, conv_c=conv_c, conv_stride=conv_stride, fc_out=10, has_bias=case % 2 == 0)
    w = WL.make_cnn_workload(f"cnn_fr{case}", 80 + case, desc, m, 1, n_r, 0.1, 1e-3, n_flip=1)
    _check(B, w)
    dev = torch.device("cuda", 0)
    mdl = B.ZenoCnnModel(w.desc, w.loss)
    args = (mdl, w.x.to(dev), w.G.contiguous().to(dev), w.features.to(dev), w.gamma, w.rho)
    out = []
    for short in (0, 0, 256):
        ws = B.alloc_workspace(mdl, m, n_r, dev)
        ws[: ws.numel() // 4 * 4].view(torch.float32).fill_(float("nan") if out else 0.0)
        out.append(npy(B.zeno_score(*args, labels=w.labels.to(dev), workspace=ws[: ws.numel() - short])))
    assert np.array_equal(out[0], out[1])
    s_ref, scale = O.cnn_scores(npy(w.x), npy(w.G), w.gamma, w.rho, w.desc, w.loss, npy(w.features), npy(w.labels))
    assert np.all(score_error(out[2], s_ref, scale) <= SCORE_TOL["fp32"])


@pytest.mark.parametrize("h,conv_c,conv_stride,m,n_r", [
    (10, [64, 64], [2, 2], 2, 3), (10, [64, 64], [2, 2], 30, 1),       # few tiles: taken, and not, the kernels outweigh their use
    (20, [64, 64], [1, 1], 12, 20), (20, [16, 24], [1, 1], 16, 20),    # large tiles: many channels, few
])
def test_cnn_on_both_sides_of_the_line_for_fragments(B, h, conv_c, conv_stride, m, n_r):
    desc = dict(in_h=h, in_w=h, in_c=3, conv_c=conv_c, conv_stride=conv_stride, fc_out=10, has_bias=True)
    _check(B, WL.make_cnn_workload("cnn_line", 100 + h, desc, m, 1, n_r, 0.1, 1e-3, seed=m, n_flip=1, worker_batch=4))


@pytest.mark.parametrize("out", [8, 9, 32, 33])
@pytest.mark.parametrize("hw,conv_c", [(5, [7]), (8, [16, 24])])
def test_cnn_widths_of_the_fully_connected_layer(B, hw, conv_c, out):
    """Up to 32 outputs its pass at x rides with the candidates' last convolution (eight outputs at a time); 175 and 1536
    columns, the former no multiple of four; gathered and staged convolutions."""
    desc = dict(in_h=hw, in_w=hw, in_c=3, conv_c=conv_c, conv_stride=[1] * len(conv_c), fc_out=out, has_bias=out != 9)
    _check(B, WL.make_cnn_workload(f"cnn_fc{out}", 120 + out, desc, 4, 1, 6, 0.1, 1e-3, n_flip=1))


@pytest.mark.parametrize("hw,conv_c", [(6, [16, 16]), (5, [9, 12])])
def test_cnn_with_as_many_candidates_as_the_calls_take(B, hw, conv_c):
    """1023 candidates, staged and gathered: every score."""
    desc = dict(in_h=hw, in_w=hw, in_c=3, conv_c=conv_c, conv_stride=[1, 2], fc_out=4, has_bias=True)
    _check(B, WL.make_cnn_workload("cnn_many", 150, desc, 1023, 300, 3, 0.1, 1e-3, n_flip=100, worker_batch=1))


@pytest.mark.parametrize("out", [8, 9])
def test_cnn_fully_connected_layer_with_a_million_columns(B, out):
    """1050625 columns of one sample: up to eight outputs beside the convolution, more in a launch of their own."""
    desc = dict(in_h=1025, in_w=1025, in_c=1, conv_c=[1], conv_stride=[1], fc_out=out, has_bias=True)
    w = WL.make_cnn_workload(f"cnn_columns{out}", 140 + out, desc, 2, 1, 1, 0.1, 1e-3, worker_batch=1)
    _check(B, w)


EDGES = [
    # (in_h, in_w, in_c, channels, strides), m, n_r
    ((9, 7, 8, [32, 33], [1, 2]), 3, 3),         # eight channels: steps of two taps; one channel beyond a tile
    ((8, 8, 17, [64, 12], [2, 1]), 3, 5),        # seventeen channels: a second unit of one channel; two channel tiles
    ((4, 4, 24, [40, 40, 8], [2, 1, 1]), 4, 9),  # a second unit of one group; 2 x 2 maps, many samples per tile
    ((1, 1, 48, [16, 16], [1, 2]), 2, 40),       # maps of one pixel
    ((6, 5, 72, [96], [1]), 2, 2),               # more units than are staged at once
    ((16, 16, 3, [32, 32, 64], [1, 2, 1]), 20, 30),   # wide tiles, one and two channel tiles
    ((15, 13, 20, [20, 64], [1, 2]), 30, 21),    # wide tiles with channels that end inside a group, the last tile cut short
    ((3, 1001, 1, [3, 2], [1, 1]), 2, 2),        # rows too wide for the staging
]


@pytest.mark.parametrize("case", range(len(EDGES)))
def test_cnn_edges_of_the_staged_tiles(B, case):
    """Every score at the fp32 tolerance at the sizes where the convolution kernels change shape: channels per unit, units
    per stage, channel tiles, position tiles that cross rows and samples, and maps that are not staged at all."""
    (h, w_, c, conv_c, conv_stride), m, n_r = EDGES[case]
    desc = dict(in_h=h, in_w=w_, in_c=c, conv_c=conv_c, conv_stride=conv_stride, fc_out=7, has_bias=case != 4)
    w = WL.make_cnn_workload(f"cnn_edge{case}", 50 + case, desc, m, 1, n_r, 0.1, 1e-3, seed=case, n_flip=1, worker_batch=4)
    _check(B, w)


@pytest.mark.parametrize("h,w_,c,conv_c,conv_stride,m,n_r", [
    (9, 7, 1, [33, 100, 5], [2, 1, 2], 5, 3),     # pass at x with more tiles than a candidate, then fewer; then none
    (8, 8, 3, [12, 64, 9], [1, 2, 1], 6, 5),      # 64 channels for the pass at x, 12 for the candidates
    (16, 16, 20, [7, 8, 31], [1, 1, 2], 9, 12),   # a first layer that is gathered: the small jobs in a launch of their own
    (32, 32, 3, [33, 16], [1, 1], 24, 6),         # staged wide tiles beside a gathered pass at x, one wave per tile after them
    (5, 5, 16, [20, 20], [1, 2], 40, 2),          # whole groups for the candidates, not for the pass at x
])
def test_cnn_channels_that_are_no_multiple_of_eight(B, h, w_, c, conv_c, conv_stride, m, n_r):
    """Every score where staged and gathered layers follow each other and share a launch with the pass at x."""
    desc = dict(in_h=h, in_w=w_, in_c=c, conv_c=conv_c, conv_stride=conv_stride, fc_out=7, has_bias=True)
    _check(B, WL.make_cnn_workload("cnn_gather", 80, desc, m, 1, n_r, 0.1, 1e-3, seed=m, n_flip=1, worker_batch=4))


RANGE = [
    # (in_h, in_w, in_c, channels, strides), m, n_r
    ((5, 6, 8, [16, 12], [1, 2]), 7, 5),           # staged, few tiles, steps of two taps
    ((16, 16, 16, [32, 8], [1, 1]), 8, 40),        # staged, many tiles
    ((5, 6, 9, [11, 12], [1, 2]), 7, 5),           # gathered
]


def _range_workload(case):
    (h, w_, c, conv_c, conv_stride), m, n_r = RANGE[case]
    desc = dict(in_h=h, in_w=w_, in_c=c, conv_c=conv_c, conv_stride=conv_stride, fc_out=3, has_bias=True)
    w = WL.make_cnn_workload("cnn_range", 70 + case, desc, m, 1, n_r, 0.1, 0.0)
    w.features.abs_().add_(0.5)
    return w, c


@pytest.mark.parametrize("case", range(len(RANGE)))
def test_cnn_infinite_kernel_values(B, case):
    """A kernel value of -inf at x (centre tap: it only meets values above zero) switches its unit off everywhere, for the pass at x
    and for every candidate; the other units' scores are finite and those of the oracle.  Where operands are split into
    pieces, the remainders of an infinite value are NaN and must not reach the sum."""
    w, c = _range_workload(case)
    w.x[:9 * c].view(9, c)[4, 3] = -float("inf")
    with np.errstate(invalid="ignore"):
        err = _check(B, w)
    assert np.all(np.isfinite(err)) and np.all(np.isfinite(npy(_gpu_scores(B, w))))


@pytest.mark.parametrize("case", range(len(RANGE)))
def test_cnn_finite_values_at_the_end_of_the_range(B, case):
    """Finite kernel values up to the largest float32, which bf16 rounds to infinity, meet zeros only (a channel of the images that
    is zero, a unit that is off): the scores are finite and those of the oracle."""
    w, c = _range_workload(case)
    (_, _, _, conv_c, _), m, n_r = RANGE[case]
    w.features.view(n_r, -1, c)[:, :, 2] = 0.0
    first = 9 * c * conv_c[0]
    w.x[first + 5] = -1e3                                       # bias: unit 5 of the first convolution is off
    big = float(np.finfo(np.float32).max)
    for i, v in ((1, big), (2, -big), (3, 3.3962e38), (4, -3.39e38)):
        w.G[i, :first].view(conv_c[0], 9, c)[0, 4, 2] = v       # meets the channel of zeros
    second = first + conv_c[0]
    for i, v in ((4, big), (5, -big), (6, 3.3962e38)):
        w.G[i, second:second + 9 * conv_c[0] * conv_c[1]].view(conv_c[1], 9, conv_c[0])[1, 4, 5] = v   # meets the unit that is off
    err = _check(B, w)
    assert np.all(np.isfinite(err))


def test_cnn_error_codes(B):
    with pytest.raises(B.ZenoError):
        B.ZenoCnnModel(dict(in_h=4, in_w=4, in_c=1, conv_c=[4], conv_stride=[3], fc_out=2, has_bias=True))
    with pytest.raises(B.ZenoError):
        B.ZenoCnnModel(dict(in_h=4, in_w=4, in_c=1, conv_c=[4], conv_stride=[1], fc_out=2, has_bias=True), "squared")
    mdl = B.ZenoCnnModel(dict(in_h=4, in_w=4, in_c=1, conv_c=[4], conv_stride=[1], fc_out=2, has_bias=True))
    assert mdl.workspace_bytes(4, 129) == 0 and mdl.workspace_bytes(4, 128) > 0
    assert mdl.plan_check(4, 4) == 2


@pytest.mark.parametrize("c,first,m,n_r", [(2, 16, 9, 30), (2, 17, 9, 30), (3, 16, 9, 30), (4, 8, 9, 30), (5, 8, 9, 30), (1, 1, 10, 33)])
def test_cnn_few_channels_in_many_tiles(B, c, first, m, n_r):
    """Both sides of the line between wide staged tiles and gathered ones for a first convolution with few channels (at least 512
    tiles of 128 positions)."""
    desc = dict(in_h=16, in_w=16, in_c=c, conv_c=[first, 8], conv_stride=[1, 2], fc_out=7, has_bias=True)
    _check(B, WL.make_cnn_workload("cnn_few", 90, desc, m, 1, n_r, 0.1, 1e-3, seed=c, n_flip=1, worker_batch=4))
