"""Percentile scales of several rows for small and large ranks, on whole and partial parts of a scale block, ragged row lengths and inputs
whose large values lie in one place, are all alike or infinite: the scales and codes are those of a sorted block."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ql():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2511_11446_amd as ql
    ql.lib()
    return ql


def _input(kind, blocks, n, g):
    x = torch.randn(blocks, n, generator=g)
    if kind == "equal":
        x = torch.full((blocks, n), -0.75)
    elif kind == "zeros but one":
        x = torch.zeros(blocks, n)
        x[:, n - 1] = 3.0
    elif kind == "large together":   # all large values next to each other, at the end of the block
        x[:, : n - 2000] *= 1e-4
    elif kind == "infinite":
        x[:, ::5] = float("inf")
    return x.half()


@pytest.mark.parametrize("rank", [1, 2, 295, 1536, 5000])
@pytest.mark.parametrize("kind", ["normal", "equal", "zeros but one", "large together", "infinite"])
@pytest.mark.parametrize("R,K", [(32, 512), (72, 512), (64, 520), (1024, 512)])
def test_scale_of_every_rank(ql, R, K, kind, rank):
    n, blocks = R * K, 3
    x = _input(kind, blocks, n, torch.Generator().manual_seed(rank))
    p_ppm = (n - rank) * 1000000 // n + 1
    k = min(n, (n * p_ppm + 999999) // 1000000)           # nearest rank: the k-th smallest magnitude
    tau = x.abs().float().sort(dim=1).values[:, k - 1]
    alpha = torch.where(tau == 0, torch.ones_like(tau), tau / 31.0)
    q, scales = ql.daq_quantize_robust(x.reshape(blocks * R, K).cuda(), R, p_ppm, 6)
    torch.testing.assert_close(scales.cpu(), alpha, rtol=0, atol=0)
    if bool(tau.isfinite().all()):
        t = tau[:, None]
        want = (x.float().clamp(-t, t) / alpha[:, None]).round().clamp(-31, 31)
        torch.testing.assert_close(q.cpu().reshape(blocks, n).float(), want, rtol=0, atol=0)


# one row per scale: ranks that are walked to from the top and ranks that are searched for, in rows of every kind of kernel; rows with fewer magnitudes than the rank
@pytest.mark.parametrize("rank", [1, 2, 3, 8, 9, 100])
@pytest.mark.parametrize("kind", ["normal", "equal", "zeros but one", "infinite"])
@pytest.mark.parametrize("K", [136, 512, 520, 1024, 1536, 2048, 4608, 8192])
def test_scale_of_a_row(ql, K, kind, rank):
    M = 70
    x = _input(kind, M, K, torch.Generator().manual_seed(rank + K))
    x[3] = 0
    x[4] = torch.arange(K).remainder(3).half()        # three magnitudes
    p_ppm = (K - rank) * 1000000 // K + 1
    k = min(K, (K * p_ppm + 999999) // 1000000)
    tau = x.abs().float().sort(dim=1).values[:, k - 1]
    alpha = torch.where(tau == 0, torch.ones_like(tau), tau / 127.0)
    q, scales = ql.daq_quantize_robust(x.cuda(), 1, p_ppm, 8)
    torch.testing.assert_close(scales.cpu(), alpha, rtol=0, atol=0)
    finite = tau.isfinite()
    t = tau[:, None]
    want = (x.float().clamp(-t, t) / alpha[:, None]).round().clamp(-127, 127)
    torch.testing.assert_close(q.cpu().float()[finite], want[finite], rtol=0, atol=0)
