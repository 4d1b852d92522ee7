"""Launches of four-wave workgroups whose tiles are all cut into K slices (too few wide tiles to fill the chip otherwise), and
uneven candidate counts in the scheduling units: every score against the oracle, the launch shapes read back."""
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


CASES = [
    # dims, m, n_r, fwd, row_align, bias
    ([3072, 512, 10], 20, 32, "fp32", 1, True),        # the pass at x rides along, sliced as well
    ([1030, 600, 300, 10], 33, 100, "bf16", 1, True),  # four row blocks, ragged K, a width that ends inside a tile
    ([960, 520, 130], 17, 40, "fp32", 32, False),      # two row blocks; 17 candidates: units of 9 and 8
    ([2048, 700], 20, 20, "fp32", 32, True),           # one layer: the pass at x is the same layer
    ([1024, 1024, 1024, 65], 12, 64, "fp32", 4, True), # second product in fp32, two row blocks; 65 outputs
    ([2048, 900, 10], 12, 150, "bf16", 32, True),      # two passes over G
    ([640, 449, 1], 30, 3, "fp32", 1, True),          # squared loss, few samples
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_sliced_layers_all_rows(B, case):
    dims, m, n_r, fwd, row_align, bias = CASES[case]
    loss = "squared" if dims[-1] == 1 else "softmax_ce"
    w = WL.make_mlp_workload(f"sliced{case}", 80 + case, dims, m, m // 3, n_r, 0.05, 1e-3, fwd, seed=case, has_bias=bias,
                             loss=loss, n_flip=m // 6, n_noise=m // 6, noise_std=2.0, worker_batch=16)
    dev = torch.device("cuda", 0)
    mdl = B.ZenoModel(w.dims, w.has_bias, w.loss, w.fwd)
    G = rows_to_gpu(B, w.G, row_align, dev)
    args = (mdl, w.x.to(dev), G, w.features.to(dev), w.gamma, w.rho)
    batch = dict(labels=None if w.labels is None else w.labels.to(dev), targets=None if w.targets is None else w.targets.to(dev))
    ws = B.alloc_workspace(mdl, m, n_r, dev)
    ws.view(torch.float32)[: ws.numel() // 4].fill_(float("nan"))   # every slot is written before it is read
    B.profile_enable(True)
    try:
        s = B.zeno_score(*args, workspace=ws, **batch)
        torch.cuda.synchronize()
        recs = B.profile_collect(detail=True)
    finally:
        B.profile_enable(False)
    wide = [r for r in recs if r["kernel"] == "layer_cand" and r["waves"] == 4]
    assert any(r["k_slices"] >= 2 and r["tail_candidates"] == m for r in wide), recs
    s_ref, scale = oracle_terms(w)
    err = score_error(npy(s), s_ref, scale)
    assert np.all(err <= SCORE_TOL[fwd]), (float(err.max()), int(err.argmax()))
    # the slices are added in slice order whoever arrives last, and the static scratch array takes the same slices
    assert torch.equal(s, B.zeno_score(*args, workspace=ws, **batch))
    if mdl.workspace_bytes(m, n_r) <= B.STATIC_SCRATCH_BYTES:
        assert torch.equal(s, B.zeno_score_static(*args, **batch))



def _shapes_and_scores(name, dims, m, n_r, fwd, row_align):
    """Launch records of the candidates' layers; every score against the oracle."""
    from paper_1805_10032_amd import binding as B
    B.load_library()
    w = WL.make_mlp_workload(name, 170 + m, dims, m, m // 3, n_r, 0.05, 1e-3, fwd, seed=m, loss="squared" if dims[-1] == 1 else
                             "softmax_ce", n_flip=m // 6, n_noise=m // 6, noise_std=2.0, worker_batch=16)
    dev = torch.device("cuda", 0)
    batch = dict(labels=None if w.labels is None else w.labels.to(dev), targets=None if w.targets is None else w.targets.to(dev))
    B.profile_enable(True)
    try:
        s = B.zeno_score(B.ZenoModel(w.dims, w.has_bias, w.loss, w.fwd), w.x.to(dev), rows_to_gpu(B, w.G, row_align, dev), w.features.to(dev),
                         w.gamma, w.rho, **batch)
        torch.cuda.synchronize()
        recs = B.profile_collect(detail=True)
    finally:
        B.profile_enable(False)
    s_ref, scale = oracle_terms(w)
    err = score_error(npy(s), s_ref, scale)
    assert np.all(err <= SCORE_TOL[fwd]), (float(err.max()), int(err.argmax()))
    return [r for r in recs if r["kernel"] == "layer_cand"]


@pytest.mark.parametrize("dims,m,n_r,fwd,row_align,waves", [
    ([512, 128], 63, 5, "fp32", 1, [1]),                 # 256 one-wave workgroups, resident all at once
    ([512, 128], 64, 5, "fp32", 1, [4]),                 # 260
    ([1000, 100], 40, 40, "bf16", 1, [1]),               # narrow output layers in bf16, packed rows
    ([900, 70], 30, 100, "bf16", 1, [1]),
    ([1500, 300], 12, 100, "bf16", 1, [1]),
    ([960, 520, 130], 17, 40, "bf16", 32, [1, 1]),       # with the pass at x, without and with the second product
    ([640, 449, 1], 30, 3, "bf16", 1, [1, 1]),
    ([320, 1600, 66], 8, 70, "fp32", 4, [1, 1]),         # the pass at x has five times the candidates' chunks, K split over waves
    ([64, 2432, 1000], 7, 100, "bf16", 1, [4, 4]),       # 38 times, without the split: 29 MB of activations copied
    ([64, 2432, 66], 7, 100, "bf16", 1, [1, 1]),         # 9 MB
    ([30, 897, 363, 244, 1], 17, 7, "bf16", 1, [1, 4, 1, 1]),   # no split for the pass at x, whose K is short: three slices
    ([1024, 600], 8, 100, "fp32", 1, [4]),               # two waves a tile, 171 tiles
    ([960, 600], 8, 100, "fp32", 1, [1]),                # 15 chunks
    ([256, 1024], 20, 70, "bf16", 1, [4]),               # short K: activations copied once per 32 features, 44 MB
    ([128, 1024], 15, 70, "bf16", 1, [1]),               # 17 MB
])
def test_one_wave_tiles_where_they_are_resident_at_once(dims, m, n_r, fwd, row_align, waves):
    """Launches on both sides of the line between one-wave tiles and four-wave workgroups: shape and every score."""
    recs = _shapes_and_scores("onewave", dims, m, n_r, fwd, row_align)
    assert [r["waves"] for r in recs] == waves, recs


@pytest.mark.parametrize("dims,m,n_r,fwd,row_align,slices,streaming", [
    ([2048, 700], 43, 33, "bf16", 1, 1, 2),              # 264 tiles, packed 16-byte aligned rows: the shifted grid
    ([2048, 702], 43, 33, "bf16", 1, 1, 3),              # 8-byte aligned
    ([2048, 700], 43, 33, "bf16", 32, 1, 1),             # line-aligned, one product in bf16
    ([1792, 700], 43, 9, "fp32", 1, 3, 0),               # 28 chunks: sliced
    ([1728, 700], 43, 9, "fp32", 1, 1, 0),               # 27
    ([1792, 512], 64, 9, "fp32", 32, 1, 1),              # the candidates fill one round exactly
    ([1792, 700], 57, 9, "fp32", 1, 1, 0),               # 348 tiles: more than 4/3 rounds
])
def test_whole_four_wave_tiles_and_their_slices(dims, m, n_r, fwd, row_align, slices, streaming):
    """Launches with 128-feature tiles for every compute unit: sliced only where their last round would be nearly empty, and not
    on the shifted column grid."""
    (r,) = _shapes_and_scores("whole", dims, m, n_r, fwd, row_align)
    assert (r["waves"], r["k_slices"], r["streaming"], r["tail_candidates"]) == (4, slices, streaming, m if slices > 1 else 0), r


@pytest.mark.parametrize("m,k_slices", [(127, 1), (128, 2), (191, 2), (192, 1)])   # 256, 258, 384, 386 tiles of 32 features
def test_two_one_wave_workgroups_per_tile(m, k_slices):
    """At most 64 features and more tiles than compute units, up to one and a half times as many: two one-wave workgroups share
    a tile, on both sides a workgroup of several waves has a tile to itself."""
    (r,) = _shapes_and_scores("two", [2048, 64], m, 5, "fp32", 1)
    assert (r["waves"], r["k_slices"]) == (1, k_slices), r
