"""DAQ kernels at the edges of their dispatch: row lengths around those that a whole workgroup takes, and channel groups on slabs of every
kind; scales and codes are those of the IEEE quotient computed on the CPU."""
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


def _check(x, amax, q, scales):
    """x fp32 and amax broadcast against each other, q and scales as the call returned them"""
    alpha = torch.where(amax == 0, torch.ones_like(amax), amax / 127.0)
    torch.testing.assert_close(scales.cpu().reshape(alpha.shape), alpha, rtol=0, atol=0)
    want = (x / alpha).round().clamp(-127, 127)
    torch.testing.assert_close(q.cpu().reshape(x.shape).float(), want, rtol=0, atol=0)


# K = 2048 and 2560: the last row lengths of four and five pieces per lane; 8192: the last one held in registers
@pytest.mark.parametrize("K", [2048, 2056, 2560, 2568, 4096, 4104, 4608, 6144, 6152, 8192, 8200])
@pytest.mark.parametrize("M", [1, 5, 130])
def test_long_rows(ql, M, K):
    x = torch.randn(M, K, generator=torch.Generator().manual_seed(K + M)).half()
    x[0] = 0
    x[M - 1, K - 1] = -57.0
    q, scales = ql.daq_quantize(x.cuda(), 1)
    _check(x.float(), x.abs().float().amax(dim=1, keepdim=True), q, scales)


@pytest.mark.parametrize("M", [8192, 8193])
def test_rows_of_five_pieces_by_count(ql, M):
    x = torch.randn(M, 2304, generator=torch.Generator().manual_seed(M)).half()
    q, scales = ql.daq_quantize(x.cuda(), 1)
    _check(x.float(), x.abs().float().amax(dim=1, keepdim=True), q, scales)


# blocks of one, a few and more than 16 slabs; slabs of 16 and 8 rows and none, codes of 8 and 16 rows per workgroup; rows side by side from one to more
# than four
@pytest.mark.parametrize("M,R", [(48, 16), (96, 24), (512, 256), (544, 272), (1024, 1024), (60, 12), (96, 96), (6400, 256), (6400, 16)])
@pytest.mark.parametrize("K,group", [(128, 32), (384, 64), (1152, 288), (1152, 32), (3072, 128), (4608, 128), (4608, 32)])
def test_channel_groups(ql, M, R, K, group):
    x = torch.randn(M, K, generator=torch.Generator().manual_seed(M + K)).half()
    x[:R, :group] = 0
    x[M - 1, K - 1] = 91.0
    q, scales = ql.daq_quantize_cg(x.cuda(), R, group)
    v = x.float().reshape(M // R, R, K // group, group)
    amax = v.abs().amax(dim=3, keepdim=True).amax(dim=1, keepdim=True)
    _check(v, amax, q.reshape(-1), scales.reshape(-1))


# whole layers with channel scales on the pipelined tiles: few groups, as many as the small table holds, one more, and the most; every group whose
# pattern is unrolled; a width at which 2048 rows take the large tiles in one round
@pytest.mark.parametrize("K,group,N", [(128, 128, 648), (1152, 288, 648), (1152, 192, 648), (1280, 32, 648), (1408, 32, 648), (1152, 64, 648), (4608, 32, 648),
                                       (768, 96, 648), (1152, 128, 3400)])
@pytest.mark.parametrize("M,R", [(256, 64), (2048, 256), (4096, 2048)])
@pytest.mark.parametrize("storage", [8, 4])
def test_layers_with_channel_scales(ql, storage, M, R, K, group, N):
    g = torch.Generator(device="cuda").manual_seed(K + M)
    x = torch.randn(M, K, device="cuda", generator=g).half()
    most = 32 if storage == 8 else 8
    w = torch.randint(-most, most, (N, K), dtype=torch.int8, device="cuda", generator=g)
    held = w if storage == 8 else torch.from_numpy(ql.ql_pack_w4_host(w.cpu().numpy())).cuda()
    s = (torch.rand(N, K // group, device="cuda", generator=g) * 0.02 + 0.001).half()
    y = ql.qlinear_grouped(x, R, held, s, group, act_group=group, storage=storage)
    q, a = ql.daq_quantize_cg(x, R, group)
    a = a.double().reshape(M // R, K // group).repeat_interleave(R, 0)
    want, scale = torch.zeros(M, N, dtype=torch.float64, device="cuda"), torch.zeros(M, N, dtype=torch.float64, device="cuda")
    for i in range(K // group):
        k = slice(i * group, (i + 1) * group)
        p = (q[:, k].double() @ w[:, k].double().T.contiguous()) * a[:, i : i + 1] * s[:, i].double()
        want += p
        scale += p.abs()
    # every group adds one rounding of its scale product and one of the running sum; then one rounding to fp16
    bound = (K // group + 3) * 2.0 ** -23 * scale + want.abs() * 2.0 ** -11 + 2.0 ** -24
    assert bool(((y.double() - want).abs() <= bound).all())


# An infinite or NaN input stays inside its scale block.  More tiles than workgroups are resident, so that a workgroup walks from a tile of one
# block to one of another: 128x128 tiles (512 resident) and 64x64 ones (768 with int8 codes, 1024 with packed ones)
@pytest.mark.parametrize("M,K,N,R,storage", [(16384, 1152, 1152, 256, 8), (16384, 768, 2304, 1024, 4), (832, 1152, 4992, 64, 8), (3200, 768, 2560, 64, 4)])
@pytest.mark.parametrize("group", [32, 64, 96, 128, 192])
def test_channel_scales_of_one_block_reach_no_other(ql, M, K, N, R, storage, group):
    g = torch.Generator(device="cuda").manual_seed(K + group)
    x = torch.randn(M, K, device="cuda", generator=g).half()
    w = torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda", generator=g)
    if storage == 4:
        w = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device="cuda", generator=g)
    s = (torch.rand(N, K // group, device="cuda", generator=g) * 0.02 + 0.001).half()
    clean = ql.qlinear_grouped(x, R, w, s, group, act_group=group, storage=storage)
    assert bool(clean.isfinite().all())
    # every third block: a walk goes on a power of two of rows further down
    bad = x.clone().reshape(M // R, R, K)
    bad[::6, R - 1, K - 1] = float("inf")
    bad[3::6, 0, K - group] = float("nan")
    y = ql.qlinear_grouped(bad.reshape(M, K), R, w, s, group, act_group=group, storage=storage).reshape(M // R, R, N)
    assert not bool(y[::3].isfinite().all())
    clean = clean.reshape(M // R, R, N)
    for i in (1, 2):
        torch.testing.assert_close(y[i::3], clean[i::3], rtol=0, atol=0)
