"""Batches of more than 128 samples: groups of 128 that share their launches, the same groups one after the other on a workspace
without room for all of them, and models that always take them one after the other; every score against the oracle."""
import numpy as np
import pytest
import torch

from paper_1805_10032_amd import workloads as WL
from tests._util import SCORE_TOL, npy, oracle_terms, rows_to_gpu, score_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,m,n_r,fwd,row_align,shared", [
    ([1001, 777, 333, 7], 33, 200, "bf16", 1, True),
    ([1001, 777, 333, 7], 30, 129, "fp32", 1, True),      # split operands: a last group of 64 rows without samples
    ([1001, 777, 333, 7], 12, 256, "fp32", 32, True),     # full groups
    ([2048, 900, 10], 12, 257, "bf16", 32, True),         # three groups, the last of one sample; K slices of wide workgroups
    ([300, 64, 1], 9, 385, "fp32", 4, True),              # four groups of one-wave tiles, squared loss
    ([64, 700], 20, 512, "bf16", 1, True),                # one layer: the pass at x rides along
    ([64, 700], 20, 513, "bf16", 1, False),               # five passes
    ([256, 1024, 10], 70, 150, "bf16", 32, False),        # eight-wave workgroups
])
def test_more_than_128_samples(dims, m, n_r, fwd, row_align, shared):
    from paper_1805_10032_amd import binding as B
    B.load_library()
    loss = "squared" if dims[-1] == 1 else "softmax_ce"
    w = WL.make_mlp_workload("passes", 400 + n_r, dims, m, m // 3, n_r, 0.05, 1e-3, fwd, seed=m, loss=loss, n_flip=m // 6,
                             n_noise=m // 6, noise_std=2.0, worker_batch=16)
    dev = torch.device("cuda", 0)
    mdl = B.ZenoModel(w.dims, w.has_bias, w.loss, w.fwd)
    G = rows_to_gpu(B, w.G, row_align, dev)
    args = (mdl, w.x.to(dev), G, w.features.to(dev), w.gamma, w.rho)
    batch = dict(labels=None if w.labels is None else w.labels.to(dev), targets=None if w.targets is None else w.targets.to(dev))
    s_ref, scale = oracle_terms(w)
    passes = (n_r + 127) // 128
    scores = []
    full = mdl.workspace_bytes(m, n_r)
    for size in (full, full - 1) if shared else (full,):
        ws = torch.full((full,), 0xff, dtype=torch.uint8, device=dev)   # NaNs: every slot is written before it is read
        B.profile_enable(True)
        try:
            s = B.zeno_score(*args, workspace=ws[:size], **batch)
            torch.cuda.synchronize()
            recs = [r for r in B.profile_collect(detail=True) if r["kernel"] == "layer_cand"]
        finally:
            B.profile_enable(False)
        assert len(recs) == (len(dims) - 1) * (1 if shared and size == full else passes), recs
        assert all(r["row_blocks"] == 4 for r in recs), recs
        err = score_error(npy(s), s_ref, scale)
        assert np.all(err <= SCORE_TOL[fwd]), (size, float(err.max()), int(err.argmax()))
        assert torch.equal(s, B.zeno_score(*args, workspace=ws[:size], **batch))
        scores.append(s)
    if len(scores) == 2:
        assert torch.equal(scores[0], scores[1])   # the groups run the same sums wherever they run
    if mdl.workspace_bytes(m, 128) + 8 * m * n_r + 4096 <= B.STATIC_SCRATCH_BYTES:
        assert torch.equal(scores[0], B.zeno_score_static(*args, **batch))


def test_a_workspace_for_one_group_at_a_time_is_enough():
    """The smallest workspace accepted holds one group's activations, whatever the batch."""
    from paper_1805_10032_amd import binding as B
    B.load_library()
    mdl = B.ZenoModel([512, 512, 10], True, "softmax_ce", "bf16")
    dev = torch.device("cuda", 0)
    d, m, n_r = mdl.num_params, 20, 256
    G, x = torch.zeros((m, d), device=dev), torch.zeros(d, device=dev)
    args = (mdl, x, G, torch.zeros((n_r, 512), device=dev), 0.1, 0.0)
    labels = torch.zeros(n_r, dtype=torch.int32, device=dev)
    one = mdl.workspace_bytes(m, 128) + 8 * m * n_r + 4096   # the loss differences of all samples besides
    assert one < mdl.workspace_bytes(m, n_r)
    ws = torch.empty(one, dtype=torch.uint8, device=dev)
    assert torch.equal(B.zeno_score(*args, labels=labels, workspace=ws), torch.zeros(m, device=dev))
    with pytest.raises(B.ZenoError):
        B.zeno_score(*args, labels=labels, workspace=ws[: one // 2])
