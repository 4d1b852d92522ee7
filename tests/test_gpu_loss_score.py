"""Loss and score in one launch (up to 16 classes and 64 samples) and in two: every score against the oracle on both sides of
the line."""
import pytest
import torch

from paper_1805_10032_amd import workloads as WL
from tests._util import SCORE_TOL, npy, oracle_terms, rows_to_gpu, score_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("classes,n_r", [(16, 64), (17, 64), (16, 65), (1, 64), (1, 1), (2, 33), (10, 130)])
def test_scores_on_both_sides_of_the_line(classes, n_r):
    from paper_1805_10032_amd import binding as B
    B.load_library()
    w = WL.make_mlp_workload(f"loss{classes}", 500 + n_r, [70, 200, classes], 9, 3, n_r, 0.05, 1e-3, "fp32", seed=classes,
                             loss="squared" if classes == 1 else "softmax_ce", n_flip=1, n_noise=1, noise_std=2.0)
    dev = torch.device("cuda", 0)
    mdl = B.ZenoModel(w.dims, w.has_bias, w.loss, w.fwd)
    batch = dict(labels=None if w.labels is None else w.labels.to(dev), targets=None if w.targets is None else w.targets.to(dev))
    s = B.zeno_score(mdl, w.x.to(dev), rows_to_gpu(B, w.G, 1, dev), w.features.to(dev), w.gamma, w.rho, **batch)
    s_ref, scale = oracle_terms(w)
    err = score_error(npy(s), s_ref, scale)
    assert (err <= SCORE_TOL["fp32"]).all(), (float(err.max()), int(err.argmax()))
