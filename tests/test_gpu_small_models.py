"""Small models, scored in one launch by a workgroup per candidate: the edges of its tiles and of the rule that takes a call
there, every score against the oracle."""
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


CASES = [
    # dims, m, n_r, fwd, row_align, bias, one launch
    ([4, 1], 3, 1, "fp32", 1, True, True),                 # shortest rows, one sample, fewer steps than waves
    ([3, 5], 3, 2, "fp32", 1, True, False),                # rows below four floats
    ([7, 16], 5, 32, "bf16", 1, False, True),              # most classes, all samples, end of a row inside a step
    ([784, 17], 4, 8, "fp32", 32, True, False),            # one class more
    ([785, 10], 9, 33, "fp32", 1, True, False),            # one sample more
    ([1000, 10], 20, 31, "fp32", 1, True, True),           # 250 steps; 1001 would be 252
    ([1001, 10], 20, 31, "fp32", 1, True, False),
    ([496, 10], 20, 31, "bf16", 1, True, True),            # 124 steps, and 126: the line for bf16 operands
    ([497, 10], 20, 31, "bf16", 1, True, False),
    ([64, 33, 10], 256, 5, "fp32", 1, True, True),         # two tiles, a workgroup for every CU
    ([64, 33, 10], 257, 5, "fp32", 1, True, False),        # one candidate more
    ([30, 32, 65, 96, 97, 1], 6, 17, "fp32", 1, True, True),   # one to four tiles, squared loss
    ([21, 128, 4, 2], 8, 32, "bf16", 4, True, True),       # widest layer, shortest hidden row
    ([50, 129, 3], 4, 3, "fp32", 1, True, False),          # one feature too wide
    ([2208, 32, 10], 5, 9, "fp32", 1, True, True),         # two layers: 564 steps, and 606 (600 is the line)
    ([2376, 32, 10], 5, 9, "fp32", 1, True, False),
    ([800, 80, 40, 32, 10], 6, 31, "fp32", 1, True, True), # four layers: 687 steps
    ([1248, 16, 10], 7, 5, "bf16", 1, True, True),         # 318 steps, and 366: the line for two layers of bf16 operands is 360
    ([1440, 16, 10], 7, 5, "bf16", 1, True, False),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_small_models_against_oracle(B, case):
    dims, m, n_r, fwd, row_align, bias, one = CASES[case]
    loss = "squared" if dims[-1] == 1 else "softmax_ce"
    w = WL.make_mlp_workload(f"small{case}", 300 + case, dims, m, m // 3, n_r, 0.05, 1e-3, fwd, seed=case, has_bias=bias,
                             loss=loss, n_flip=m // 6, n_noise=m // 6, noise_std=2.0, worker_batch=16)
    dev = torch.device("cuda", 0)
    mdl = B.ZenoModel(w.dims, w.has_bias, w.loss, w.fwd)
    args = (mdl, w.x.to(dev), rows_to_gpu(B, w.G, row_align, dev), w.features.to(dev), w.gamma, w.rho)
    batch = dict(labels=None if w.labels is None else w.labels.to(dev), targets=None if w.targets is None else w.targets.to(dev))
    B.profile_enable(True)
    try:
        s = B.zeno_score(*args, **batch)
        torch.cuda.synchronize()
        recs = B.profile_collect(detail=True)
    finally:
        B.profile_enable(False)
    assert (len(recs) == 1) == one, recs
    s_ref, scale = oracle_terms(w)
    err = score_error(npy(s), s_ref, scale)
    assert (err <= SCORE_TOL[fwd]).all(), (float(err.max()), int(err.argmax()))
    assert torch.equal(s, B.zeno_score_static(*args, **batch))


def test_small_model_labels_out_of_range_and_padding(B):
    """A label outside the classes makes every score NaN; infinite entries of one candidate stay with it."""
    dev = torch.device("cuda", 0)
    w = WL.make_mlp_workload("small_inf", 400, [20, 40, 6], 5, 1, 7, 0.05, 1e-3, "fp32", seed=3)
    mdl = B.ZenoModel(w.dims, w.has_bias, w.loss, w.fwd)
    G = w.G.clone()
    G[1, 19] = float("inf")                    # last weight of a row, beside another row's
    G[3, -1] = float("nan")
    labels = w.labels.to(dev)
    call = lambda g, lab: npy(B.zeno_score(mdl, w.x.to(dev), rows_to_gpu(B, g, 1), w.features.to(dev), w.gamma, w.rho, labels=lab))
    clean, s = call(w.G, labels), call(G, labels)
    assert not (s[1] > -float("inf")) and s[3] != s[3]
    assert (s[[0, 2, 4]] == clean[[0, 2, 4]]).all()
    bad = labels.clone()
    bad[2] = 6
    s = call(w.G, bad)
    assert (s != s).all()
