"""CPU-only checks of the C-ABI library: it loads, exports what the header declares,
rejects bad arguments before touching a device, and its host helpers work."""
import ctypes
import os
import re

import numpy as np
import pytest

import paper_2511_11446_amd as ql
import workload

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "diffpro_qlinear.h")


def _declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = re.findall(r"\b([a-z_0-9]+)\s*\([^;{]*\)\s*;", text)
    return sorted(set(n for n in names if n not in ("defined",)))


def test_library_loads_and_exports_every_declared_symbol():
    L = ql.lib()
    declared = _declared_functions()
    assert len(declared) >= 19
    for name in declared:
        assert hasattr(L, name), name
    assert sorted(declared) == sorted(ql.EXPORTS)
    assert L.ql_version() >= 1000
    assert L.ql_status_string(0) == b"QL_OK" and L.ql_status_string(5) == b"QL_ERR_WORKSPACE"
    assert L.ql_num_gemm_variants() >= 4
    assert all(ql.gemm_variants())


FAKE = ctypes.c_void_p(0x1000)       # never dereferenced: every call below must fail validation first
FAKE_ODD = ctypes.c_void_p(0x1001)


def test_daq_argument_checks():
    L = ql.lib()
    assert L.daq_quantize(None, 4, 8, 1, FAKE, FAKE, None, 0, None) == 1
    assert L.daq_quantize(FAKE, 4, 8, 1, None, FAKE, None, 0, None) == 1
    assert L.daq_quantize(FAKE, 0, 8, 1, FAKE, FAKE, None, 0, None) == 2
    assert L.daq_quantize(FAKE, 4, 0, 1, FAKE, FAKE, None, 0, None) == 2
    assert L.daq_quantize(FAKE, 6, 8, 4, FAKE, FAKE, None, 0, None) == 2          # M % R != 0
    assert L.daq_quantize(FAKE, 4, 133144, 1, FAKE, FAKE, None, 0, None) == 2      # K too long for int32 sums
    assert L.daq_quantize(FAKE_ODD, 4, 8, 1, FAKE, FAKE, None, 0, None) == 3
    assert L.daq_quantize(FAKE, 8, 8, 4, FAKE, FAKE, None, 0, None) == 5           # R > 1 needs a workspace
    assert L.daq_quantize(FAKE, 8, 8, 4, FAKE, FAKE, FAKE, 4, None) == 5           # too small
    assert L.daq_quantize(FAKE, 8, 8, 4, FAKE, FAKE, ctypes.c_void_p(0x1010), 4096, None) == 3  # not 256-aligned
    assert ql.daq_workspace_bytes(8, 8, 1) == 0 and ql.daq_workspace_bytes(8, 8, 4) >= 8


def test_qlinear_argument_checks():
    L = ql.lib()
    big = 1 << 30
    for fn in (L.qlinear_w8a8, L.qlinear_w4a8):
        assert fn(None, 4, 128, 1, FAKE, FAKE, None, 8, FAKE, None, FAKE, big, None) == 1
        assert fn(FAKE, 4, 128, 1, None, FAKE, None, 8, FAKE, None, FAKE, big, None) == 1
        assert fn(FAKE, 4, 128, 1, FAKE, None, None, 8, FAKE, None, FAKE, big, None) == 1
        assert fn(FAKE, 4, 128, 1, FAKE, FAKE, None, 8, None, None, FAKE, big, None) == 1
        assert fn(FAKE, 4, 128, 1, FAKE, FAKE, None, 0, FAKE, None, FAKE, big, None) == 2
        assert fn(FAKE, 4, 128, 3, FAKE, FAKE, None, 8, FAKE, None, FAKE, big, None) == 2
        assert fn(FAKE, 4, 128, 1, FAKE, FAKE, None, 8, FAKE, None, None, 0, None) == 5
        assert fn(FAKE, 4, 128, 1, FAKE, FAKE, None, 8, FAKE, None, FAKE, 16, None) == 5
        assert fn(FAKE, 4, 128, 1, FAKE, FAKE_ODD, None, 8, FAKE, None, FAKE, big, None) == 3
        assert fn(FAKE, 1 << 20, 1 << 12, 1, FAKE, FAKE, None, 8, FAKE, None, FAKE, big, None) == 2  # M*K >= 2^31
    # 4-bit weights need whole groups of 128
    assert L.qlinear_w4a8(FAKE, 4, 192, 1, FAKE, FAKE, None, 8, FAKE, None, FAKE, big, None) == 2
    assert L.qgemm_w4a8(FAKE, FAKE, 4, 192, 1, FAKE, FAKE, None, 8, FAKE, None, None) == 2
    assert L.qgemm_w8a8(None, FAKE, 4, 128, 1, FAKE, FAKE, None, 8, FAKE, None, None) == 1
    assert L.qgemm_w8a8(FAKE, FAKE, 4, 128, 1, FAKE, FAKE, None, 8, FAKE, FAKE_ODD, None) == 3
    assert ql.qlinear_workspace_bytes(16, 128, 1) >= 16 * 128 + 16 * 4
    assert ql.qlinear_workspace_bytes(16, 128, 4) > ql.qlinear_workspace_bytes(16, 128, 16) - 512


def test_plan_argument_checks():
    L = ql.lib()
    h = ctypes.c_void_p()

    def desc(K=1152, N=1152, bits=8, group=0, w=0x1000, s=0x2000, b=0):
        return ql.ql_layer_desc(K, N, bits, group, w, s, b)

    arr = (ql.ql_layer_desc * 2)(desc(), desc(bits=4, group=128))
    assert L.ql_plan_create(arr, 2, 256, ctypes.byref(h)) == 0 and h.value
    assert L.ql_plan_num_layers(h) == 2
    assert L.ql_plan_workspace_bytes(h, 256, 1) >= 256 * 1152
    assert L.ql_plan_workspace_bytes(h, 512, 1) == 0          # beyond M_max
    xs = (ctypes.c_void_p * 2)(0x1000, 0x1000)
    ys = (ctypes.c_void_p * 2)(0x1000, 0)
    assert L.qlinear_plan_run(h, xs, ys, 256, 1, FAKE, 1 << 30, None) == 1   # a NULL output
    ys = (ctypes.c_void_p * 2)(0x1000, 0x1000)
    assert L.qlinear_plan_run(h, xs, ys, 512, 1, FAKE, 1 << 30, None) == 2   # M > M_max
    assert L.qlinear_plan_run(h, xs, ys, 256, 7, FAKE, 1 << 30, None) == 2   # M % R
    assert L.qlinear_plan_run(h, xs, ys, 256, 1, FAKE, 64, None) == 5
    assert L.qlinear_plan_run(None, xs, ys, 256, 1, FAKE, 1 << 30, None) == 1
    L.ql_plan_destroy(h)
    bad = [(desc(bits=6), 4), (desc(bits=8, group=128), 4), (desc(bits=4, group=0), 4), (desc(bits=4, group=48), 4),
           (desc(K=1100, bits=4, group=128), 2), (desc(w=0), 1), (desc(s=0), 1), (desc(N=0), 2), (desc(s=0x2001), 3)]
    for d, want in bad:
        arr = (ql.ql_layer_desc * 1)(d)
        assert L.ql_plan_create(arr, 1, 256, ctypes.byref(h)) == want
        assert not h.value
    assert L.ql_plan_create(arr, 0, 256, ctypes.byref(h)) == 2
    assert L.ql_plan_create(None, 1, 256, ctypes.byref(h)) == 1


def test_plan_workspace_covers_every_layer():
    """The widest layer of a plan does not always need the most: with K % 8 != 0 it has no partial maxima, and a narrower layer's
    then reached behind the workspace."""
    L = ql.lib()
    h = ctypes.c_void_p()
    for Ks, M, R in [((8193, 8192), 8192, 8192), ((1152, 4608), 16384, 256), ((4609, 4608, 1152), 16384, 16384), ((40, 33), 64, 8)]:
        arr = (ql.ql_layer_desc * len(Ks))(*[ql.ql_layer_desc(K, 64, 8, 0, 0x1000, 0x2000, 0) for K in Ks])
        assert L.ql_plan_create(arr, len(Ks), M, ctypes.byref(h)) == 0
        assert L.ql_plan_workspace_bytes(h, M, R) == max(ql.qlinear_workspace_bytes(M, K, R) for K in Ks)
        L.ql_plan_destroy(h)


def test_variant_override_range():
    L = ql.lib()
    n = L.ql_num_gemm_variants()
    assert L.ql_set_gemm_variant(n + 1) == 4 and L.ql_set_gemm_variant(-2) == 4
    assert L.ql_set_gemm_variant(n) == 0      # n selects the generic kernel
    assert L.ql_set_gemm_variant(-1) == 0


def test_pack_w4_host_matches_documented_order(orc):
    # hand-derived from the storage rule: byte j of a run of 8 holds k=j (low) and k=4+j (high)
    w = np.array([[0, 1, 2, 3, 4, 5, 6, 7, -8, -7, -6, -5, -4, -3, -2, -1]], np.int8)
    assert ql.ql_pack_w4_host(w).tolist() == [[0x40, 0x51, 0x62, 0x73, 0xC8, 0xD9, 0xEA, 0xFB]]
    codes = workload.w4_codes(33, 256, "abi")
    packed = ql.ql_pack_w4_host(codes)
    # the oracle's independent packer and unpacker agree with the library's host packer
    assert np.array_equal(packed, orc.pack_w4(codes))
    assert np.array_equal(orc.unpack_w4(packed, 256), codes)
    bad = codes.copy()
    bad[3, 7] = 8
    with pytest.raises(ql.QlError):
        ql.ql_pack_w4_host(bad)


def test_workload_recipe_is_deterministic():
    a = workload.activations(8, 1152, "det", 3)
    b = workload.activations(8, 1152, "det", 3)
    assert np.array_equal(a.view(np.uint16), b.view(np.uint16))
    assert not np.array_equal(a, workload.activations(8, 1152, "det", 4))
    ch = workload.outlier_channels(1152, 8, "det", 3)
    assert len(set(ch.tolist())) == 8
    assert np.abs(a[:, ch].astype(np.float32)).mean() > 5 * np.abs(a.astype(np.float32)).mean() / 2
    plan = workload.bit_plan()
    assert len(plan) == 112 and all(p["bits"] == 8 for p in plan[:12] + plan[-12:])
    n4 = sum(p["bits"] == 4 for p in plan)
    assert 60 <= n4 <= 88 and plan == workload.bit_plan()
    s = workload.sigma_schedule(25)
    assert abs(s[0] - 5.0) < 1e-12 and abs(s[-1] - 0.2) < 1e-12 and np.all(np.diff(s) < 0)


def test_daq_division_free_codes_exhaustive(tmp_path):
    """The kernels' division-free quantization equals the division of eq. (4) on every (threshold, value) fp16 pair
    that passes its near-tie test (the rest take the division), for every code width 2..8 bits (q_max = 1 ... 127);
    checked on the host, all 5e8 pairs per width."""
    import subprocess
    src = os.path.join(os.path.dirname(__file__), "daq_division_free_check.c")
    exe = str(tmp_path / "daq_check")
    subprocess.run(["gcc", "-O2", "-ffp-contract=off", "-fopenmp", "-o", exe, src, "-lm"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    lines = [l for l in r.stdout.splitlines() if l.startswith("qmax")]
    assert [int(l.split()[1]) for l in lines] == [127, 63, 31, 15, 7, 3, 1]
    assert all("mismatches 0 out-of-range 0" in l for l in lines), r.stdout


def test_split_k_walk_stays_inside_the_row_and_the_lds(tmp_path):
    """The few-rows kernel's walk over K, from the kernel's own header: every slice once, nothing read behind the row or behind the
    LDS that holds the workgroup's codes, for every inner size up to 5120 and every weight group."""
    import subprocess
    exe = str(tmp_path / "split_walk_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-o", exe, os.path.join(os.path.dirname(__file__), "split_walk_check.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


def test_split_k_walk_on_eight_wavefronts(tmp_path):
    """The same on eight wavefronts, and the LDS slots of the rings."""
    import subprocess
    exe = str(tmp_path / "split_wide_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-o", exe, os.path.join(os.path.dirname(__file__), "split_wide_check.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


def test_pieces_of_rows_that_are_no_whole_steps_stay_inside_their_row(tmp_path):
    """Addresses of the DMA tiles for any K, from the kernel's own header, up to the largest operands that the entry points accept."""
    import subprocess
    exe = str(tmp_path / "dma_piece_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-o", exe, os.path.join(os.path.dirname(__file__), "dma_piece_check.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.fixture(scope="module")
def plan_windows(tmp_path_factory):
    """(M, R, p_ppm, a_bits, room, [(K, N, bits, group, x, y)]) -> [(first layer, layers, {those whose GEMMs share a launch})], from the library's own decision."""
    import subprocess
    exe = str(tmp_path_factory.mktemp("plan_window") / "check")
    here = os.path.dirname(os.path.abspath(__file__))
    lib = os.path.join(os.path.dirname(here), "paper_2511_11446_amd", "libdiffpro_qlinear.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-o", exe,
                    os.path.join(here, "plan_window_check.cpp"), lib, "-Wl,-rpath," + os.path.dirname(lib)], check=True)

    def ask(M, R, p_ppm, a_bits, room, layers, *one_round):
        text = "%d %d %d %d %d\n" % (M, R, p_ppm, a_bits, room) + "".join("%d %d %d %d %d %d\n" % l for l in layers)
        r = subprocess.run([exe, *one_round], input=text, capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr
        out = []
        for line in r.stdout.splitlines():
            head, _, together = line.partition(":")
            first, n = map(int, head.split())
            out.append((first, n, set(map(int, together.split()))))
        return out
    return ask


def _place(buffer, element=0):
    """A made-up address: buffers of up to 8 GiB, far apart."""
    return (1 << 40) + (buffer << 33) + 2 * element


def test_every_kind_of_layer_takes_part_in_a_shared_gemm_launch(plan_windows):
    """The plans that the GPU tests run bring every kind of tile into the launch that several layers share."""
    import test_gpu_plan_windows as pw
    kinds = set()
    for shapes in pw.PLANS.values():
        for M in pw.ROWS:
            for room in pw.ROOM:
                layers = [(K, N, bits, group, _place(2 * i), _place(2 * i + 1)) for i, (K, N, bits, group, _) in enumerate(shapes)]
                for _, _, together in plan_windows(M, 1, 0, 8, room, layers):
                    kinds |= {(shapes[i][2], shapes[i][3]) for i in together}
    assert kinds >= {(8, 0), (16, 0), (4, 32), (4, 64), (4, 128), (4, 192), (4, 288)}


def test_4_bit_layers_of_more_small_tiles_than_cus_share_a_gemm_launch(plan_windows):
    """A 4-bit projection that would split K by itself goes with its neighbours where it is more than one 32x32 tile per CU, as long as it has more groups than wavefronts."""
    def taken(M, group):
        shapes = [(768, 2304, 8, 0), (768, 768, 4, group), (768, 3072, 8, 0)]
        (_, _, together), = plan_windows(M, 1, 0, 8, 4, [s + (_place(2 * i), _place(2 * i + 1)) for i, s in enumerate(shapes)])
        return 1 in together
    assert [taken(M, 128) for M in (320, 321, 325, 602, 682)] == [False, True, True, True, True]
    assert not taken(325, 192)      # four groups


def test_one_round_of_large_tiles(plan_windows):
    """Rows and layers of the GPU test: 256 large tiles at most, all taken; one row tile more, short rows, a 4-bit layer, an output not in whole pieces: none."""
    import test_gpu_plan_windows as pw

    def taken(M, shapes, R=1):
        layers = [(K, N, bits, group, _place(2 * i), _place(2 * i + 1)) for i, (K, N, bits, group, _) in enumerate(shapes)]
        (_, _, together), = plan_windows(M, R, 0, 8, 4, layers, "one round")
        return together

    for name, M, R in pw.ROUNDS:
        assert taken(M, pw.ROUND_LAYERS[name], R) == set(range(len(pw.ROUND_LAYERS[name]))), (name, M, R)
    block = pw.ROUND_LAYERS["block"]
    assert not taken(2049, block)
    assert not taken(2048, [(256,) + l[1:] for l in block])
    assert not taken(2048, block[:2] + [(1152, 4608, 4, 128, True)])
    assert not taken(2048, block[:2] + [(1152, 4604, 8, 0, True)])


def test_layers_that_wait_for_each_other_share_no_gemm_launch(plan_windows):
    import test_gpu_plan_windows as pw
    want = {
        "disjoint": [(0, 4, {0, 1, 2, 3})],
        "one output": [(0, 4, set())],
        "outputs five rows apart": [(0, 4, set())],
        "outputs that meet": [(0, 4, {0, 1, 2, 3})],
        "an output that a later layer reads": [(2, 2, {2, 3})],     # layers 0 and 1: one of them quantized
        "an output over the input of an earlier FP16 layer": [(0, 4, set())],
        "an output over the last rows of an FP16 input": [(0, 4, set())],
        "an output over the input of an earlier 8-bit layer": [(0, 4, {0, 1, 2, 3})],   # which is quantized before any GEMM
    }
    assert set(want) == set(pw.ALIASES)
    for name, (xs, ys) in pw.ALIASES.items():
        layers = [(K, N, bits, group, _place(*x), _place(*y)) for (K, N, bits, group, _), x, y in zip(pw.ALIAS_LAYERS, xs, ys)]
        assert plan_windows(pw.ALIAS_M, 1, 0, 8, 4, layers) == want[name], name


def test_room_and_size_of_a_window(plan_windows):
    """Layers go together as far as their codes fit the workspace, at most eight, and as far as codes and earlier outputs stay within 256 MB."""
    def windows(M, shapes, room, R=1, p_ppm=0):
        return plan_windows(M, R, p_ppm, 8, room, [(K, N, 8, 0, _place(2 * i), _place(2 * i + 1)) for i, (K, N) in enumerate(shapes)])
    sizes = lambda w: [(first, n) for first, n, _ in w]
    # the recommended workspace is the widest layer's: three layers of a quarter of its width, and none of equal width
    assert sizes(windows(2048, [(1152, 3456), (1152, 1152), (1152, 4608), (4608, 1152)], 1)) == [(0, 3)]
    assert sizes(windows(2048, [(1152, 1152)] * 4, 1)) == []
    assert sizes(windows(2048, [(1152, 1152)] * 4, 2)) == [(0, 2), (2, 2)]
    assert sizes(windows(2048, [(384, 1152)] * 10, 10)) == [(0, 8), (8, 2)]
    # 65536 rows: 75 MB of codes and 151 MB of outputs per layer
    assert sizes(windows(65536, [(1152, 1152)] * 4, 4)) == []
    assert sizes(windows(16384, [(1152, 3456), (1152, 1152), (1152, 4608)], 3)) == [(0, 3)]
    # percentiles: up to 4096 scale blocks
    assert sizes(windows(8192, [(384, 1152)] * 2, 2, R=2, p_ppm=750000)) == [(0, 2)]
    assert sizes(windows(8194, [(384, 1152)] * 2, 2, R=2, p_ppm=750000)) == []


class _Prm(ctypes.Structure):
    _fields_ = [("p_ppm", ctypes.c_int32), ("a_bits", ctypes.c_int32)]


def test_robust_daq_argument_checks_and_time_bins():
    L = ql.lib()
    ok = _Prm(999000, 8)
    assert L.daq_quantize_robust(FAKE, 4, 8, 1, None, FAKE, FAKE, None, 0, None) == 1
    assert L.daq_quantize_robust(None, 4, 8, 1, ctypes.byref(ok), FAKE, FAKE, None, 0, None) == 1
    assert L.daq_quantize_robust(FAKE, 6, 8, 4, ctypes.byref(ok), FAKE, FAKE, None, 0, None) == 2
    for bad in (_Prm(0, 8), _Prm(1000001, 8), _Prm(999000, 1), _Prm(999000, 9)):
        assert L.daq_quantize_robust(FAKE, 4, 8, 1, ctypes.byref(bad), FAKE, FAKE, None, 0, None) == 4
    assert L.daq_quantize_robust(FAKE, 8, 8, 4, ctypes.byref(ok), FAKE, FAKE, None, 0, None) == 5
    assert L.qlinear_plan_run_robust(None, None, None, 4, 1, ctypes.byref(ok), None, 0, None) == 1
    # equal thirds of the schedule, in sampling order
    assert [ql.time_bin(i, 6) for i in range(6)] == [0, 0, 1, 1, 2, 2]
    assert [ql.time_bin(i, 25) for i in (0, 8, 9, 16, 17, 24)] == [0, 0, 1, 1, 2, 2]
    assert ql.time_bin(-1, 5) == -1 and ql.time_bin(5, 5) == -1 and ql.time_bin(0, 0) == -1


def test_group_size_argument_checks():
    L = ql.lib()
    ws = ctypes.c_void_p(0x10000)
    big = 1 << 30
    args = lambda K, g: (FAKE, 4, K, 1, FAKE, FAKE, g, None, 8, FAKE, None, ws, big, None)
    assert L.qlinear_w4a8_g(*args(1152, 48)) == 4       # not a multiple of 32
    assert L.qlinear_w4a8_g(*args(1152, 0)) == 4
    assert L.qlinear_w4a8_g(*args(1152, 320)) == 2      # does not divide K
    assert L.qlinear_w4a8_g(*args(100, 100)) == 4
    assert L.qgemm_w4a8_g(FAKE, FAKE, 4, 1152, 1, FAKE, FAKE, 48, None, 8, FAKE, None, None) == 4
    assert L.qgemm_w4a8_g(FAKE, FAKE, 4, 1152, 1, FAKE, FAKE, 256, None, 8, FAKE, None, None) == 2
    # a group whose sum of 127 * 8 * 16 products could pass 2^31 is refused; the largest admitted one is 132096
    assert L.qlinear_w4a8_g(*args(132224, 132224)) == 2
    assert 127 * 128 * 132096 < 2 ** 31 <= 127 * 128 * 132128


def test_fused_epilogue_argument_checks():
    L = ql.lib()
    ws = ctypes.c_void_p(0x10000)
    big = 1 << 30
    def call(fu, M=8):
        return L.qlinear_w8a8_fused(FAKE, M, 64, 1, FAKE, FAKE, None, 8, ctypes.byref(fu) if fu else None, FAKE, ws, big, None)
    assert call(ql.ql_fusion(7, 0, None, None, 1)) == 4                       # unknown activation
    assert call(ql.ql_fusion(0, 0, 0x1001, None, 1)) == 3                     # odd residual pointer
    assert call(ql.ql_fusion(0, 0, None, 0x1000, 3)) == 2                     # M % gate_rows
    assert call(ql.ql_fusion(0, 0, None, 0x1000, 0)) == 2
    assert L.qlinear_w4a8_fused(FAKE, 8, 1152, 1, FAKE, FAKE, 48, None, 8, None, FAKE, ws, big, None) == 4   # bad group


def test_fp16_layer_argument_checks():
    L = ql.lib()
    assert L.qlinear_f16(None, 4, 8, FAKE, None, 8, None, FAKE, None) == 1
    assert L.qlinear_f16(FAKE, 4, 8, FAKE_ODD, None, 8, None, FAKE, None) == 3
    assert L.qlinear_f16(FAKE, 0, 8, FAKE, None, 8, None, FAKE, None) == 2
    h = ctypes.c_void_p()
    d = ql.ql_layer_desc(64, 8, 16, 0, 0x1000, 0, 0)
    assert L.ql_plan_create((ql.ql_layer_desc * 1)(d), 1, 16, ctypes.byref(h)) == 0     # FP16 layer: no scales needed
    L.ql_plan_destroy(h)
    d = ql.ql_layer_desc(64, 8, 16, 128, 0x1000, 0, 0)
    assert L.ql_plan_create((ql.ql_layer_desc * 1)(d), 1, 16, ctypes.byref(h)) == 4     # groups belong to 4-bit layers


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    """No fallback: without the built HIP library every entry point of the binding raises."""
    monkeypatch.setattr(ql, "_lib", None)
    monkeypatch.setattr(ql, "LIB_PATH", str(tmp_path / "libdiffpro_qlinear.so"))
    with pytest.raises(ImportError, match="no fallback"):
        ql.lib()
    with pytest.raises(ImportError):
        ql.daq_workspace_bytes(8, 8, 4)


def test_repack_from_pair_order_equals_packing_the_codes(orc):
    g = workload.rng("repack")
    w = g.integers(-8, 8, size=(5, 64), dtype=np.int8)
    pairs = ((w[:, 0::2] & 0xF) | ((w[:, 1::2] & 0xF) << 4)).astype(np.uint8)      # low nibble = even k, high nibble = odd k
    got = ql.ql_repack_w4_pairs_host(pairs)
    assert np.array_equal(got, ql.ql_pack_w4_host(w))
    assert np.array_equal(orc.unpack_w4(got, 64), w)
    L = ql.lib()
    buf = pairs.ctypes.data_as(ctypes.c_void_p)
    assert L.ql_repack_w4_pairs_host(buf, 5, 64, buf) == 4          # in place
    assert L.ql_repack_w4_pairs_host(buf, 5, 60, buf) in (2, 4)
    assert L.ql_repack_w4_pairs_host(None, 5, 64, buf) == 1


def test_daq_quantize_rowmax_argument_checks():
    L = ql.lib()
    x, rm, q, sc, ws = (ctypes.c_void_p(v) for v in (0x10000, 0x20000, 0x30000, 0x40000, 0x50000))
    assert L.daq_quantize_rowmax(x, 64, 128, 1, None, q, sc, None, 0, None) == 1          # no row maxima
    assert L.daq_quantize_rowmax(x, 64, 128, 1, ctypes.c_void_p(0x20002), q, sc, None, 0, None) == 3
    assert L.daq_quantize_rowmax(x, 64, 128, 5, rm, q, sc, ws, 1 << 20, None) == 2        # M % R
    assert L.daq_quantize_rowmax(x, 64, 128, 32, rm, q, sc, None, 0, None) == 5           # workspace for R > 1
    fu = ql.ql_fusion(0, 0, None, None, 1, 0x1002)                                        # misaligned side output
    assert L.qlinear_w8a8_fused(x, 64, 128, 1, rm, sc, None, 64, ctypes.byref(fu), q, ws, 1 << 20, None) == 3


def test_prepack_w4_argument_checks():
    """The device-side re-layout validates before any device call (fake, aligned pointers)."""
    L = ql.lib()
    a, b = ctypes.c_void_p(0x10000), ctypes.c_void_p(0x20000)
    assert L.ql_prepack_w4(None, 5, 64, b, None) == 1
    assert L.ql_prepack_w4(a, 5, 64, None, None) == 1
    assert L.ql_prepack_w4(a, 5, 64, a, None) == 4                  # in place
    assert L.ql_prepack_w4(a, 5, 60, b, None) == 2                  # K % 8
    assert L.ql_prepack_w4(a, 0, 64, b, None) == 2
    assert L.ql_prepack_w4(ctypes.c_void_p(0x10002), 5, 64, b, None) == 3


def test_layernorm_daq_argument_checks():
    L = ql.lib()
    fn = L.daq_quantize_ln
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64,
                   ctypes.c_float, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    A = ctypes.c_void_p(0x10000)
    assert fn(None, 8, 64, 1, None, None, 1, 1e-6, None, A, A, None, 0, None) == 1
    assert fn(A, 8, 64, 1, None, None, 1, 1e-6, None, None, None, None, 0, None) == 1      # nothing to produce
    assert fn(A, 8, 64, 1, None, None, 1, 1e-6, None, A, None, None, 0, None) == 1          # codes without scales
    assert fn(ctypes.c_void_p(0x10008), 8, 64, 1, None, None, 1, 1e-6, None, A, A, None, 0, None) == 3
    assert fn(A, 8, 60, 1, None, None, 1, 1e-6, None, A, A, None, 0, None) == 2             # K % 8
    assert fn(A, 8, 4616, 1, None, None, 1, 1e-6, None, A, A, None, 0, None) == 2           # longer than the register row
    assert fn(A, 8, 64, 1, A, None, 3, 1e-6, None, A, A, None, 0, None) == 2                # M % rows_per_mod
    assert fn(A, 8, 64, 4, None, None, 1, 1e-6, None, A, A, None, 0, None) == 1             # R > 1 needs h
    assert fn(A, 8, 64, 4, None, None, 1, 1e-6, A, A, A, None, 0, None) in (0, 5, 6)        # shape ok: workspace or device next


def test_plan_space_host_helpers_and_argument_checks(orc):
    g = np.random.default_rng(5)
    for b in (3, 6, 2, 7):
        c = g.integers(-(1 << (b - 1)), 1 << (b - 1), (4, 64), dtype=np.int8)
        p = ql.pack_bits_host(c, b)
        assert np.array_equal(p, orc.pack_bits(c, b))                 # the same documented storage on both sides
        assert np.array_equal(ql.unpack_bits_host(p, b, 64), c)
    with pytest.raises(ql.QlError):
        ql.pack_bits_host(np.full((1, 8), 4, np.int8), 3)            # 4 is not a 3-bit code
    with pytest.raises(ql.QlError):
        ql.pack_bits_host(np.zeros((1, 5), np.int8), 3)              # 15 bits: not whole bytes
    # asymmetric codes and zero points (as the GPTQ packer returns them: both shifted by 2^(b-1)) -> code - zero
    codes = np.array([[-8, 7, 0, -3]], np.int8)
    zeros = np.array([[-2, 5]], np.int32)
    assert ql.zero_point_fold_host(codes, zeros, 2).tolist() == [[-6, 9, -5, -8]]
    with pytest.raises(ql.QlError):
        ql.zero_point_fold_host(np.array([[-128, 127]], np.int8), np.array([[100]], np.int32), 2)
    L = ql.lib()
    A = ctypes.c_void_p(0x10000)
    L.daq_quantize_cg.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p,
                                  ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    assert L.daq_quantize_cg(A, 8, 64, 4, 12, A, A, A, 1 << 20, None) == 4       # not a multiple of 8
    assert L.daq_quantize_cg(A, 8, 64, 4, 24, A, A, A, 1 << 20, None) == 2       # does not divide K
    assert L.daq_quantize_cg(A, 8, 64, 4, 16, A, A, None, 0, None) == 5
    L.qlinear_grouped.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p,
                                  ctypes.c_int32, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p,
                                  ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    call = lambda ag, st, grp: L.qlinear_grouped(A, 128, 256, 128, ag, A, st, A, grp, None, 64, A, None, A, 1 << 24, None)
    assert call(0, 5, 128) == 4          # storage must be 4 or 8
    assert call(64, 8, 128) == 4         # channel groups must be the weight groups
    assert call(0, 8, 48) == 4           # group not a multiple of 32
    assert call(0, 8, 96) == 2           # group does not divide K
