"""More rows than one launch of the candidates' pass takes (8 threads a row up to 192 dimensions,
fewer than 2^32 threads a launch: 2^29 rows): one call over all of them against calls over four
views, whose launches are single ones.  Two dimensions keep the rows at 4.3 GB; the workspace
takes about 57 GB."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROWS, VIEW = (1 << 29) + 77, 1 << 27


@pytest.fixture(scope="module")
def many():
    import torch
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(11)
    mu = torch.tensor([[-6.0, 0.0], [5.0, 4.0], [4.0, -5.0]], device=dev)
    x = torch.empty(ROWS, 2, device=dev)
    for a in range(0, ROWS, VIEW):
        v = x[a:a + VIEW]
        v.normal_(generator=g)
        v.add_(mu[torch.randint(0, 3, (v.shape[0],), generator=g, device=dev, dtype=torch.uint8)
               .int()])
    # the last row stands alone: a call that loses the rows past a launch's end shows there
    x[-1] = torch.tensor([1e3, -1e3], device=dev)
    th = (torch.tensor([0.2, 0.3, 0.5], device=dev), mu, torch.full((3, 2), 1.5, device=dev))
    yield x, th
    del x
    torch.cuda.empty_cache()


def test_estep(many):
    import torch
    import paper_2606_10896_amd as gmm
    x, th = many
    ws = gmm.workspace(ROWS, 2, 3)

    def stats(rows):
        out = [torch.zeros(s, dtype=torch.float64, device=x.device) for s in (3, (3, 2), (3, 2), 1)]
        for a in range(0, ROWS, rows):
            gmm.gmm_estep_accumulate(x[a:a + rows], *th, *out, ws)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out]

    whole, views = stats(ROWS), stats(VIEW)
    # every point is listed (at most 3 components), so that its terms are the same in both;
    # fp64 sums of up to 2^29 terms in another order: 2^29 2^-53 at most, of the largest |sum|
    for a, b in zip(whole, views):
        assert np.abs(a - b).max() <= 2.0 ** -24 * np.abs(b).max()
    assert abs(whole[0].sum() - ROWS) <= 1e-6 * ROWS
    print(f"  N_k {whole[0]}", flush=True)


def test_assignment(many):
    import torch
    import paper_2606_10896_amd as gmm
    x, th = many
    ws = gmm.workspace(ROWS, 2, 3, 1)
    idx = torch.full((ROWS, 1), -7, dtype=torch.int32, device=x.device)
    resp = torch.full((ROWS, 1), -7.0, device=x.device)
    gmm.gmm_assign_topk(x, *th, 1, 0.0, idx, resp, ws)
    for a in range(0, ROWS, VIEW):
        v = x[a:a + VIEW]
        vi, vr = torch.empty_like(idx[:v.shape[0]]), torch.empty_like(resp[:v.shape[0]])
        gmm.gmm_assign_topk(v, *th, 1, 0.0, vi, vr, ws)
        assert bool((vi == idx[a:a + VIEW]).all()) and bool((vr == resp[a:a + VIEW]).all()), a
    assert int(idx.min()) >= 0
