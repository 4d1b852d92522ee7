"""GPU parity of zeno_aggregate / zeno_mean / zeno_median against the CPU oracle.

Integer work (the selected index set) and the three aggregators must match
bit for bit: the kernels sum the selected rows in ascending index order in fp64
and round once, exactly as the oracle does."""
import numpy as np
import pytest
import torch

from oracle import zeno_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1805_10032_amd import binding
    binding.load_library()
    return binding


def _rand_G(m, d, seed, scale=1.0):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(m, d, generator=g, dtype=torch.float32) * scale


SHAPES = [(1, 1), (1, 5), (2, 3), (3, 4), (5, 1023), (8, 64), (20, 7850), (7, 4099), (64, 10001),
          (100, 5002), (33, 65537), (128, 777), (1024, 130)]


@pytest.mark.parametrize("m,d", SHAPES)
def test_aggregate_bit_exact(B, m, d):
    G = _rand_G(m, d, 100 * m + d)
    rng = np.random.default_rng(m * 7 + d)
    scores = rng.normal(size=m).astype(np.float32)
    Gd = G.cuda()
    for b in sorted({0, m // 3, m - 1}):
        out, sel = B.zeno_aggregate(Gd, torch.from_numpy(scores).cuda(), b)
        torch.cuda.synchronize()
        ref, ref_sel = O.zeno_aggregate(G.numpy(), scores, b)
        assert np.array_equal(sel.cpu().numpy().astype(np.int64), ref_sel), (m, d, b)
        assert np.array_equal(out.cpu().numpy(), ref.astype(np.float32)), (m, d, b)


def test_aggregate_b0_equals_mean_kernel(B):
    G = _rand_G(20, 7850, 5).cuda()
    s = torch.randn(20).cuda()
    out, _ = B.zeno_aggregate(G, s, 0)
    assert torch.equal(out, B.zeno_mean(G))


def test_selection_ties_nan_and_infinities(B):
    scores = np.array([1.0, 2.0, 2.0, np.nan, 2.0, -np.inf, np.inf, -0.0, 0.0, np.nan], dtype=np.float32)
    m = len(scores)
    G = _rand_G(m, 37, 1)
    for b in range(m):
        out, sel = B.zeno_aggregate(G.cuda(), torch.from_numpy(scores).cuda(), b)
        ref, ref_sel = O.zeno_aggregate(G.numpy(), scores, b)
        assert sel.cpu().numpy().tolist() == ref_sel.tolist(), b
        assert np.array_equal(out.cpu().numpy(), ref.astype(np.float32))


def test_identical_colluding_rows_and_selected_null(B):
    """All faulty rows equal (Section 6.4): ties between them are broken by index."""
    G = _rand_G(10, 515, 2)
    G[3] = G[7] = G[8] = G[1]
    scores = torch.randn(10)
    scores[3] = scores[7] = scores[8] = scores[1]
    for b in (1, 2, 3, 8):
        out, sel = B.zeno_aggregate(G.cuda(), scores.cuda(), b, want_selected=False)
        assert sel is None
        ref, _ = O.zeno_aggregate(G.numpy(), scores.numpy(), b)
        assert np.array_equal(out.cpu().numpy(), ref.astype(np.float32))


def test_rows_only_four_byte_aligned(B):
    """d mod 4 != 0 and a base pointer that is only 4-byte aligned."""
    m, d = 9, 1001
    flat = torch.randn(m * d + 3, generator=torch.Generator().manual_seed(3)).cuda()
    for shift in (1, 2, 3):
        G = flat[shift:shift + m * d].view(m, d)
        assert G.data_ptr() % 16 != 0
        scores = torch.randn(m, generator=torch.Generator().manual_seed(4))
        out_buf = torch.empty(d + 1, device="cuda")[1:]
        out, sel = B.zeno_aggregate(G, scores.cuda(), 3, out=out_buf)
        ref, ref_sel = O.zeno_aggregate(G.cpu().numpy(), scores.numpy(), 3)
        assert np.array_equal(out.cpu().numpy(), ref.astype(np.float32))
        assert np.array_equal(B.zeno_mean(G).cpu().numpy(), O.mean(G.cpu().numpy()).astype(np.float32))
        assert np.array_equal(B.zeno_median(G).cpu().numpy(), O.median(G.cpu().numpy()).astype(np.float32))


@pytest.mark.parametrize("m,d", [(1, 7), (2, 9), (3, 100), (4, 5), (7, 4099), (8, 64), (20, 7850), (21, 1000),
                                 (33, 2049), (64, 3001), (100, 5002), (127, 300), (128, 515),
                                 # more than 128 rows: the median by rank selection in LDS
                                 (129, 300), (130, 31), (200, 1000), (255, 64), (256, 4099), (513, 777), (1000, 2049),
                                 (1023, 33), (1024, 130)])
def test_mean_and_median_bit_exact(B, m, d):
    G = _rand_G(m, d, 31 * m + d, scale=3.0)
    Gd = G.cuda()
    assert np.array_equal(B.zeno_mean(Gd).cpu().numpy(), O.mean(G.numpy()).astype(np.float32))
    med = B.zeno_median(Gd).cpu().numpy()
    assert np.array_equal(med, O.median(G.numpy()).astype(np.float32))


@pytest.mark.parametrize("row_align", [1, 32])
def test_median_every_m(B, row_align):
    """Every number of candidates the median accepts: each has its own count of compile-time and
    run-time padding keys (and the small ones the four-column lanes when the rows are aligned);
    d = 263 leaves a ragged tail behind the four-column part.  NaN and infinite entries included."""
    from tests._util import rows_to_gpu
    d = 263
    for m in range(1, 129):
        G = _rand_G(m, d, 5000 + m, scale=2.0)
        G[m // 2, ::17] = float("inf")
        G[0, 5::29] = float("nan")
        G[m - 1, 3::31] = float("-inf")
        med = B.zeno_median(rows_to_gpu(B, G, row_align)).cpu().numpy()
        ref = O.median(G.numpy()).astype(np.float32)
        assert np.array_equal(np.isnan(med), np.isnan(ref)), m
        ok = ~np.isnan(ref)
        assert np.array_equal(med[ok], ref[ok]), m


@pytest.mark.parametrize("row_align", [1, 32])
@pytest.mark.parametrize("m", [129, 192, 500, 1024])
def test_median_by_selection_with_ties_and_nonfinite_entries(B, m, row_align):
    """m > 128: ties (few distinct values, so the two middle keys are often equal), columns of one value,
    NaN, +inf and -inf entries, a column that is NaN in more than half of its rows; dense and line-aligned rows."""
    from tests._util import rows_to_gpu
    d = 333
    g = torch.Generator().manual_seed(7000 + m)
    G = torch.randint(-3, 4, (m, d), generator=g).to(torch.float32) * 0.5
    G[:, 1::4] = _rand_G(m, d, 7100 + m)[:, 1::4]
    G[:, 2] = 1.25
    G[m // 3, ::13] = float("inf")
    G[m // 2, 4::17] = float("-inf")
    G[1, 6::19] = float("nan")
    G[: m // 2 + 2, 8] = float("nan")
    G[: m // 2 + 2, 9] = float("inf")
    G[: m // 2, 10] = float("-inf")
    G[m // 2:, 10] = float("inf")
    med = B.zeno_median(rows_to_gpu(B, G, row_align)).cpu().numpy()
    ref = O.median(G.numpy()).astype(np.float32)
    assert np.array_equal(np.isnan(med), np.isnan(ref))
    ok = ~np.isnan(ref)
    assert np.array_equal(med[ok], ref[ok])


@pytest.mark.parametrize("m", [1, 2, 7, 20, 33, 100, 128, 129, 300, 513, 1024])
def test_median_keeps_the_sign_of_zero(B, m):
    """-0 sorts below +0 whatever the other columns hold: columns of zeros of either sign with the middle on either side of the
    line between them, alone and around other values, beside columns that the search for m > 128 finds in other ways."""
    d = 192
    g = torch.Generator().manual_seed(8000 + m)
    U = torch.rand((m, d), generator=g)
    X = torch.randn((m, d), generator=g)
    zero = torch.where(torch.rand((m, d), generator=g) < torch.linspace(0.3, 0.7, d), -0.0, 0.0)
    G = X.clone()
    for kind, part in ((0, 1.1), (1, 0.6), (2, 0.2), (3, 0.05)):            # share of zeros in the column
        cols = torch.arange(d) % 6 == kind
        G[:, cols] = torch.where(U < part, zero, X)[:, cols]
    G[:, 4::12] = torch.round(X * 2)[:, 4::12]                               # few values, zeros of either sign among them
    G[m // 2:, 0::24] = float("nan")
    G[m // 2, 1::30] = float("inf")
    v = np.sort(G.numpy(), axis=0)                                           # NaN last; the zeros of a column in any order
    n = (G.numpy() < 0).sum(0) + ((G.numpy() == 0) & np.signbit(G.numpy())).sum(0)
    k = (m - 1) // 2
    def at(r):
        return np.where(v[r] == 0, np.where(r < n, np.float32(-0.0), np.float32(0.0)), v[r]).astype(np.float64)
    ref = (at(k) if m & 1 else 0.5 * (at(k) + at(k + 1))).astype(np.float32)
    med = B.zeno_median(G.cuda()).cpu().numpy()
    ok = ~np.isnan(ref)
    assert np.array_equal(np.isnan(med), ~ok)
    assert np.array_equal(med[ok].view(np.int32), ref[ok].view(np.int32))


@pytest.mark.parametrize("m,d", [(129, 1), (160, 65), (161, 63), (288, 64), (289, 129), (320, 200), (321, 33), (384, 31),
                                 (385, 32), (575, 97), (833, 64), (960, 5), (961, 70), (1023, 257), (1024, 1)])
def test_median_by_selection_at_the_edges_of_its_tiles(B, m, d):
    """m > 128, sizes around the widths at which the kernel's keys per lane, lanes per column and columns per tile
    change; columns whose search is led astray: values over hundreds of binades, a block of equal rows around
    the middle, mostly zeros of either sign, adjacent floats, NaN in all rows but a few."""
    G = _rand_G(m, d, 9000 + m, scale=1.0)
    kind = torch.arange(d) % 6
    G[:, kind == 1] = torch.sign(G[:, kind == 1]) * torch.exp(25.0 * G[:, kind == 1])
    G[m // 4: m // 2 + 1, kind == 2] = 0.125
    G[:, kind == 3] *= (G[:, kind == 3] > 1.0)
    G[:, kind == 4] = 1.0 + torch.randint(0, 3, (m, d), generator=torch.Generator().manual_seed(m))[:, kind == 4] * 2.0 ** -23
    G[3:, kind == 5] = float("nan")
    med = B.zeno_median(G.cuda()).cpu().numpy()
    ref = O.median(G.numpy()).astype(np.float32)
    assert np.array_equal(np.isnan(med), np.isnan(ref))
    ok = ~np.isnan(ref)
    assert np.array_equal(med[ok], ref[ok])


@pytest.mark.parametrize("m", [129, 130, 200, 300, 321, 512, 700, 1024])
def test_median_by_selection_of_few_values(B, m):
    """m > 128, columns of few to some hundred values, the same kind for all columns of a wave: the lanes' medians agree in all, most
    or few columns, on values with many copies or some; the middle inside a block of equal values and at its edges."""
    kinds = [0.25, 0.5, 1.0, 2.0, 4.0, 8.0, 16.0, 32.0, 64.0]
    d = 64 * len(kinds)
    g = torch.Generator().manual_seed(8500 + m)
    G = torch.randn((m, d), generator=g)
    for i, q in enumerate(kinds):
        cols = slice(64 * i, 64 * i + 64)
        G[:, cols] = torch.round(G[:, cols] * q) / q
        G[:, 64 * i + 32: 64 * i + 64] *= 0.1 + torch.rand(32, generator=g)    # a scale of its own, as quantised gradients have
    G[m // 3, 5::37] = float("nan")
    G[: m // 2 + 1, 64 * 3 + 3] = 0.5                                          # a block that ends at the middle, and next to it
    G[: (m + 1) // 2, 64 * 4 + 4] = -3.0
    G[: m // 2, 64 * 5 + 5] = 100.0
    med = B.zeno_median(G.cuda()).cpu().numpy()
    assert np.array_equal(med, O.median(G.numpy()).astype(np.float32), equal_nan=True)


@pytest.mark.parametrize("m,d", [(130, 524_388), (320, 262_500), (1024, 66_000)])
def test_median_by_selection_over_many_tiles(B, m, d):
    """m > 128, more tiles than one generation of workgroups takes: every column near a multiple of 32 Ki columns and a random
    choice of the others; clustered rows with a colluding block, so that waves mix columns found by their lists with others."""
    g = torch.Generator(device="cuda").manual_seed(m)
    G = torch.randn((m, d), generator=g, device="cuda") * 0.02 + torch.randn(d, generator=g, device="cuda") * 0.01
    G[m // 8: m // 4] = -4.0 * G[m // 4:].mean(0)
    G[m // 2, ::4099] = float("nan")
    med = B.zeno_median(G)
    edges = torch.arange(0, d, 32768)[:, None] + torch.arange(-40, 40)
    cols = torch.cat([edges.flatten(), torch.randint(0, d, (5000,), generator=torch.Generator().manual_seed(m))]).clamp(0, d - 1)
    ref = O.median(G[:, cols.cuda()].cpu().numpy()).astype(np.float32)
    assert np.array_equal(med.cpu().numpy()[cols.numpy()], ref, equal_nan=True)


@pytest.mark.parametrize("d", [1023, 1025, 4 * 163840 - 1, 4 * 163840 + 5])
def test_average_on_both_sides_of_the_columns_per_thread(B, d):
    """One column of four floats a thread below 163840 of them, four from there on: bit for bit, with a b that leaves a batch of
    rows incomplete; the update as well."""
    m, b, gamma = 13, 4, float(np.float32(0.1))            # (the call takes a float32)
    G = _rand_G(m, d, 77 + d, scale=2.0)
    scores, x = torch.randn(m, generator=torch.Generator().manual_seed(d)), _rand_G(1, d, 78 + d)[0]
    out, sel = B.zeno_aggregate(G.cuda(), scores.cuda(), b)
    ref, ref_sel = O.zeno_aggregate(G.numpy(), scores.numpy(), b)
    assert np.array_equal(out.cpu().numpy(), ref.astype(np.float32)) and np.array_equal(sel.cpu().numpy(), ref_sel)
    assert np.array_equal(B.zeno_mean(G.cuda()).cpu().numpy(), O.mean(G.numpy()).astype(np.float32))
    x_next, _, _ = B.zeno_aggregate_update(G.cuda(), scores.cuda(), b, gamma, x.cuda())
    assert np.array_equal(x_next.cpu().numpy(), O.zeno_update(x.numpy(), G.numpy(), scores.numpy(), b, gamma)[0].astype(np.float32))


def test_median_with_nonfinite_entries(B):
    m, d = 6, 200
    G = _rand_G(m, d, 9)
    G[0, ::3] = float("nan")
    G[1, ::5] = float("inf")
    G[2, ::7] = float("-inf")
    G[3, ::2] = float("nan")
    G[4, 1::2] = -0.0
    med = B.zeno_median(G.cuda()).cpu().numpy()
    ref = O.median(G.numpy()).astype(np.float32)
    assert np.array_equal(np.isnan(med), np.isnan(ref))
    ok = ~np.isnan(ref)
    assert np.array_equal(med[ok], ref[ok])


def test_error_codes(B):
    G = torch.zeros(4, 8, device="cuda")
    s = torch.zeros(4, device="cuda")
    for bad_b in (-1, 4, 9):
        with pytest.raises(B.ZenoError) as e:
            B.zeno_aggregate(G, s, bad_b, want_selected=False)
        assert e.value.status == 1
    big = torch.zeros(1025, 8, device="cuda")     # more candidates than any call accepts
    with pytest.raises(B.ZenoError) as e:
        B.zeno_median(big)
    assert e.value.status == 1
    with pytest.raises(ValueError):
        B.zeno_mean(torch.zeros(4, 8))          # host tensor: no silent CPU path
