"""The average's column blocks: of full width, and narrower ones where these give every compute unit as many workgroups.  Sizes on both
sides of one block per compute unit, of a unit of 64 float4 columns, of a block and of a burst; every column bit for bit the float64
average."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 3, 255, 256, 257, 655359, 655360, 1048575, 1048576, 1048580, 1048833, 1578506, 2097152, 2097413,
                               4194304, 6291457, 10485763])
@pytest.mark.parametrize("m", [1, 7])
def test_every_column(d, m):
    from paper_1805_10032_amd import binding as B
    B.load_library()
    dev = torch.device("cuda", 0)
    gen = torch.Generator(device="cuda").manual_seed(d + m)
    G = torch.randn((m, d), generator=gen, device=dev)
    x = torch.randn(d, generator=gen, device=dev)
    scores = torch.randn(m, generator=gen, device=dev)
    b = m // 3

    def average(rows):
        total = torch.zeros(d, dtype=torch.float64, device=dev)
        for i in rows:
            total += G[i]
        return total / len(rows)

    guarded = torch.full((d + 64,), 7.0, device=dev)   # nothing is written behind the last column
    assert torch.equal(B.zeno_mean(G, out=guarded[:d]), average(range(m)).float())
    assert torch.equal(guarded[d:], torch.full((64,), 7.0, device=dev))
    rows = sorted(torch.argsort(scores, descending=True, stable=True)[:m - b].tolist())
    gamma = float(torch.tensor(0.1, dtype=torch.float32))
    x_ref = (x.double() - gamma * average(rows)).float()
    x_next, out, selected = B.zeno_aggregate_update(G, scores, b, 0.1, x)
    assert selected.tolist() == rows
    assert torch.equal(out, average(rows).float()) and torch.equal(x_next, x_ref)
    x_next, _, _ = B.zeno_aggregate_update(G, scores, b, 0.1, x, x_next=x, want_out=False)   # in place
    assert torch.equal(x_next, x_ref)
