"""CPU-side checks of the C-ABI library: it loads, exports every symbol the
header declares, and its argument checks reject bad calls before touching the
GPU.  No compute call is made here."""
import ctypes
import os
import re

import pytest

from paper_2307_09782_amd import zqfp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    syms = set()
    for name in sorted(os.listdir(os.path.join(ROOT, "include"))):
        text = open(os.path.join(ROOT, "include", name)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        syms |= set(re.findall(r"\b(zqfp_\w+)\s*\(", text))
    return sorted(syms)


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(zqfp.LIB_PATH):
        from paper_2307_09782_amd.build import build_lib
        build_lib()
    return zqfp.lib()


def test_header_declares_the_four_calls_of_the_boundary():
    syms = _declared_symbols()
    for name in ("zqfp_quantize_act_fp8", "zqfp_pack_weight_fp4", "zqfp_w4a8_gemm", "zqfp_w4a8_gemm_lorc"):
        assert name in syms


def test_library_exports_every_declared_symbol(lib):
    for name in _declared_symbols():
        assert hasattr(lib, name), name
    assert lib.zqfp_version() >= 100


def test_packed_size_and_shape_limits(lib):
    # codes K*N/2 + exponents K/G*N + column scales 4N, plus header and padding
    K, N, G = 4096, 12288, 128
    n = lib.zqfp_packed_weight_bytes(K, N, G)
    payload = K * N // 2 + (K // G) * N + 4 * N
    assert payload + 256 <= n <= payload + 256 + 3 * 256
    assert lib.zqfp_packed_weight_bytes(4096, 100, 128) > 0      # N need not be a multiple of 16
    assert lib.zqfp_packed_weight_bytes(4000, 128, 128) == 0     # K % 128
    assert lib.zqfp_packed_weight_bytes(4096, 128, 48) == 0      # G % 32
    assert lib.zqfp_packed_weight_bytes(4096, 128, 96) == 0      # K % G
    assert lib.zqfp_packed_weight_bytes(3200, 128, 320) > 0      # the paper's LLaMA-3b group size
    assert lib.zqfp_packed_weight_bytes(32768, 128, 32) == 0     # K / G > 256
    assert lib.zqfp_packed_weight_bytes(4096, 128, 256) > 0
    assert lib.zqfp_packed_weight_bytes(4096, 128, 32) > 0
    assert lib.zqfp_gemm_workspace_bytes(16, 4096, 4096) == 0


def test_argument_checks_return_error_codes_without_a_gpu(lib):
    p = ctypes.c_void_p
    buf = (ctypes.c_uint8 * 4096)()
    a = ctypes.addressof(buf)
    a16 = (a + 255) // 256 * 256
    # quantizer: K % 128, NULL pointers, alignment
    assert lib.zqfp_quantize_act_fp8(p(a16), 1, 100, 100, p(a16), p(a16), None, 0, None, None) == -2
    assert lib.zqfp_quantize_act_fp8(None, 1, 128, 128, p(a16), p(a16), None, 0, None, None) == -1
    assert lib.zqfp_quantize_act_fp8(p(a16 + 2), 1, 128, 128, p(a16), p(a16), None, 0, None, None) == -3
    assert lib.zqfp_quantize_act_fp8(p(a16), 1, 128, 128, p(a16), p(a16), None, 8, None, None) == -1
    assert lib.zqfp_quantize_act_fp8(p(a16), 0, 128, 128, p(a16), p(a16), None, 0, None, None) == 0
    # packer: mode, shape
    assert lib.zqfp_pack_weight_fp4(p(a16), 128, 16, 16, 128, 3, p(a16), None) == -4
    assert lib.zqfp_pack_weight_fp4(p(a16), 128, 16, 8, 128, 1, p(a16), None) == -2
    assert lib.zqfp_pack_weight_fp4(p(a16), 128, 16, 16, 128, 1, None, None) == -1
    assert lib.zqfp_pack_weight_fp4(p(a16), 128, 16, 16, 128, 1, p(a16 + 16), None) == -3
    # gemm: out dtype, rank, empty problem is a no-op
    assert lib.zqfp_w4a8_gemm(p(a16), p(a16), 1, 128, p(a16), 16, 128, p(a16), 16, 7, 0, None, 0, None) == -4
    assert lib.zqfp_w4a8_gemm(p(a16), p(a16), 1, 128, p(a16), 16, 128, p(a16), 16, 0, 5, None, 0, None) == -4
    assert lib.zqfp_w4a8_gemm(p(a16), p(a16), 0, 128, p(a16), 16, 128, p(a16), 16, 0, 0, None, 0, None) == 0
    assert lib.zqfp_w4a8_gemm(p(a16), p(a16), 1, 128, None, 16, 128, p(a16), 16, 0, 0, None, 0, None) == -1
    assert lib.zqfp_w4a8_gemm(p(a16), p(a16), 1, 128, p(a16), 16, 128, p(a16), 8, 0, 0, None, 0, None) == -2
    assert lib.zqfp_w4a8_gemm_lorc(p(a16), p(a16), 1, 128, p(a16), 16, 128, None, None, 8, p(a16), 16, 0, 0, None, 0, None) == -1
    assert lib.zqfp_w4a8_gemm_lorc(p(a16), p(a16), 1, 128, p(a16), 16, 128, p(a16), p(a16), 65, p(a16), 16, 0, 0, None, 0, None) == -2
    # a workspace that is given must be as large as the query says (here: one 64 x 128 tile, K split 4 ways)
    need = lib.zqfp_gemm_workspace_bytes(64, 4096, 128)
    assert need > 0
    assert lib.zqfp_w4a8_gemm(p(a16), p(a16), 64, 4096, p(a16), 128, 128, p(a16), 128, 0, 0, p(a16), need - 1, None) == -6
    assert b"workspace" in lib.zqfp_last_hip_error()
    assert lib.zqfp_w4a8_gemm(p(a16), p(a16), 16, 28672, p(a16), 8192, 128, p(a16), 8192, 0, 0, p(a16), 1 << 20, None) == -6
    # shape limits of the layout itself
    assert lib.zqfp_packed_weight_bytes(128 * 4096, 16, 128 * 16) == 0   # 4096 k-tiles: beyond the limit
    assert lib.zqfp_packed_weight_bytes(128 * 4095, 16, 128 * 21) > 0


def test_packed_weight_check_reads_a_host_copy_of_the_header(lib):
    """Header fields as the packer writes them (magic 'ZQF4', version, K, N, Np, G, Gs, mode, ngs, ngq, code width,
    four section offsets): accepted for its own (K, N, G), refused for any other and after any damage."""
    import struct
    K, N, G = 512, 200, 64
    total = lib.zqfp_packed_weight_bytes(K, N, G)
    Np = 208
    off_codes = 256
    off_exps = off_codes + Np * K // 2
    ngs = K // 64
    ngq = (ngs + 3) // 4
    off_cs = (off_exps + (Np // 16) * ngq * 64 + 255) // 256 * 256
    assert total == (off_cs + 4 * Np + 255) // 256 * 256
    hdr = struct.pack("<IIqqqiiiiiIQQQQ", 0x3446515A, 1, K, N, Np, G, 64, 2, ngs, ngq, 4, off_codes, off_exps, off_cs, total)
    hdr = hdr + bytes(256 - len(hdr))
    chk = lambda h, k, n, g: lib.zqfp_packed_weight_check(h, k, n, g)
    assert chk(hdr, K, N, G) == 0
    assert chk(hdr, K, N, 128) == -7 and chk(hdr, K, N + 1, G) == -7 and chk(hdr, 2 * K, N, G) == -7
    assert chk(hdr, K, N, 48) == -2 and chk(None, K, N, G) == -1
    assert chk(b"\0" * 256, K, N, G) == -7
    for pos in (0, 4, 8, 16, 32, 40, 52, 56, 80):
        bad = bytearray(hdr)
        bad[pos] ^= 1
        assert chk(bytes(bad), K, N, G) == -7, pos


def test_binding_refuses_sizes_the_library_must_take_on_trust():
    """The wrappers compare what the C side cannot (it never reads device memory on the host): blob size against
    (K, N, G), workspace size against the query, the output's shape, dtype and row contiguity."""
    import torch
    K, N, G, M = 4096, 128, 128, 64
    nb = zqfp.packed_weight_bytes(K, N, G)
    ok = dict(M=M, K=K, N=N, G=G, packed_numel=nb, workspace_numel=None, out_shape=(M, N), out_dtype=torch.float32,
              out_stride=(N, 1))
    zqfp.check_gemm_args(**ok)
    zqfp.check_gemm_args(**{**ok, "workspace_numel": zqfp.gemm_workspace_bytes(M, K, N)})
    zqfp.check_gemm_args(**{**ok, "out_stride": (N + 8, 1), "out_dtype": torch.bfloat16})
    for change, code in (({"packed_numel": nb - 256}, -2), ({"G": 256}, -2), ({"N": 144}, -2), ({"G": 48}, -2),
                         ({"workspace_numel": zqfp.gemm_workspace_bytes(M, K, N) - 4}, -6),
                         ({"out_dtype": torch.float16}, -4), ({"out_shape": (M, N + 1)}, -2),
                         ({"out_stride": (N, 2)}, -2), ({"out_stride": (N - 1, 1)}, -2), ({"out_is_cuda": False}, -2)):
        with pytest.raises(zqfp.ZqfpError) as e:
            zqfp.check_gemm_args(**{**ok, **change})
        assert e.value.code == code, change


def test_build_rejects_spills_in_hand_scheduled_kernels():
    """The tiled GEMM waits for its LDS reads by count; the build refuses a compile in which that
    kernel uses scratch memory (a spill could save a register whose read is still in flight)."""
    from paper_2307_09782_amd import build
    ok = ("x.hip:1:1: remark: Function Name: _ZN4zqfp11k_gemm_tileILi4EEEv [-Rpass-analysis=kernel-resource-usage]\n"
          "x.hip:1:1: remark:     ScratchSize [bytes/lane]: 0 [-Rpass-analysis=kernel-resource-usage]\n"
          "x.hip:1:1: remark:     VGPRs Spill: 0 [-Rpass-analysis=kernel-resource-usage]\n"
          "x.hip:1:1: remark: Function Name: _ZN4zqfp13k_gemm_decodeILi8EEEv [-Rpass-analysis=kernel-resource-usage]\n"
          "x.hip:1:1: remark:     ScratchSize [bytes/lane]: 96 [-Rpass-analysis=kernel-resource-usage]\n")
    build._check_no_scratch(ok)  # other kernels may use scratch
    bad = ok.replace("ScratchSize [bytes/lane]: 0", "ScratchSize [bytes/lane]: 24")
    with pytest.raises(RuntimeError):
        build._check_no_scratch(bad)


def test_build_rejects_spills_in_the_register_fed_gemm():
    from paper_2307_09782_amd import build
    spilled = ("x.hip:1:1: remark: Function Name: _ZN4zqfp10k_gemm_midILi4ELi4ELi2ELb0ELi8EEEv [-Rpass-analysis=kernel-resource-usage]\n"
               "x.hip:1:1: remark:     ScratchSize [bytes/lane]: 20 [-Rpass-analysis=kernel-resource-usage]\n")
    with pytest.raises(RuntimeError):
        build._check_no_scratch(spilled)


def test_build_rejects_scratch_memory_in_gptq():
    """The remarks of the 48-channel instance with its sums in registers, and with a part of them behind a run-time index."""
    from paper_2307_09782_amd import build
    ok = ("x.hip:1:1: remark: Function Name: _ZN4zqfp12_GLOBAL__N_16k_gptqILi3ELi1EEEvPKtlPKf [-Rpass-analysis=kernel-resource-usage]\n"
          "x.hip:1:1: remark:     ScratchSize [bytes/lane]: 0 [-Rpass-analysis=kernel-resource-usage]\n"
          "x.hip:1:1: remark:     VGPRs Spill: 0 [-Rpass-analysis=kernel-resource-usage]\n")
    build._check_no_scratch(ok)
    for bad in (ok.replace("lane]: 0", "lane]: 80"), ok.replace("Spill: 0", "Spill: 4")):
        with pytest.raises(RuntimeError):
            build._check_no_scratch(bad)


def test_build_rejects_quantizers_that_leave_room_for_fewer_waves():
    """The remarks of the sums-of-sixteen quantizer as they are, and with what a few registers more would make of them."""
    from paper_2307_09782_amd import build
    ok = ("x.hip:1:1: remark: Function Name: _ZN4zqfp12_GLOBAL__N_114k_quantize_actILi16ELi256ELi1EEEvPKtll [-Rpass-analysis=kernel-resource-usage]\n"
          "x.hip:1:1: remark:     ScratchSize [bytes/lane]: 0 [-Rpass-analysis=kernel-resource-usage]\n"
          "x.hip:1:1: remark:     Occupancy [waves/SIMD]: 5 [-Rpass-analysis=kernel-resource-usage]\n"
          "x.hip:1:1: remark: Function Name: _ZN4zqfp12_GLOBAL__N_114k_quantize_actILi16ELi1024ELi1EEEvPKtll [-Rpass-analysis=kernel-resource-usage]\n"
          "x.hip:1:1: remark:     Occupancy [waves/SIMD]: 4 [-Rpass-analysis=kernel-resource-usage]\n")
    build._check_waves(ok)
    for bad in (ok.replace("SIMD]: 5", "SIMD]: 4"), ok.replace("lane]: 0", "lane]: 8")):
        with pytest.raises(RuntimeError):
            build._check_waves(bad)


def test_workspace_query_is_pure_host_logic():
    """zqfp_gemm_workspace_bytes plans on the host (no GPU needed): zero for every benchmark
    configuration, [slices][M][Np] floats where K is split."""
    lib = zqfp.lib()
    ws = lambda M, K, N: int(lib.zqfp_gemm_workspace_bytes(M, K, N))
    for (M, K, N) in [(16, 256, 256), (2048, 2048, 8192), (1, 4096, 12288), (16, 4096, 12288), (256, 4096, 12288),
                      (4096, 4096, 12288), (4096, 4096, 11008), (16, 5120, 13824), (2048, 5120, 13824),
                      (1, 8192, 28672), (4, 8192, 28672), (16, 8192, 28672), (64, 8192, 28672)]:
        assert ws(M, K, N) == 0, (M, K, N)
    assert ws(64, 4096, 128) == 4 * 64 * 128 * 4          # one tile, 32 k-tiles: 4 slices of 8
    assert ws(64, 11008, 4096) == 10 * 64 * 4096 * 4      # 32 tiles, 86 k-tiles: 10 slices of 9
    assert ws(100, 3072, 136) == 3 * 100 * 144 * 4        # Np = 144
    assert ws(16, 28672, 8192) == 4 * 16 * 8192 * 4       # decode form: 224 k-tiles in 4 chunks
    assert ws(8, 8192, 4096) == 0 and ws(0, 4096, 4096) == 0 and ws(64, 4100, 4096) == 0


def test_bench_refuses_more_than_one_gpu():
    """The build runs on one GPU: `bench.py --gpus 2` exits with a message before it touches a device."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=300)
    assert r.returncode != 0 and "ONE GPU" in r.stderr


@pytest.mark.parametrize("fp8", [False, True])
def test_sizes_that_are_no_integers_stay_refused_after_an_equal_integer(lib, fp8):
    """The binding keeps blob sizes by (K, N, G); 4096.0 equals 4096 as a key and is no size."""
    query = zqfp._blob_bytes_fp8 if fp8 else zqfp.packed_weight_bytes
    assert query(4096, 1024, 128) > 0
    for args in ((4096.0, 1024, 128), (4096, 1024.0, 128), (4096, 1024, 128.0)):
        with pytest.raises(ctypes.ArgumentError):
            query(*args)


D, M_, T, S = zqfp.FORM_DECODE, zqfp.FORM_MID, zqfp.FORM_TILE, zqfp.FORM_STREAM


@pytest.mark.parametrize("wbits,M,K,N,r,accum,form", [
    # one pass, or a low-rank correction: the tiled kernel gains more from the first and loses less to the second
    (4, 24, 8192, 28672, 0, 0, M_), (4, 24, 8192, 28672, 0, 1, T), (4, 32, 8192, 28672, 8, 0, T), (4, 17, 6144, 24576, 4, 1, T),
    (4, 32, 3072, 20000, 8, 0, T), (4, 32, 3072, 20000, 0, 1, T), (4, 64, 4096, 12288, 8, 1, M_),
    # K beyond 16384 rows
    (4, 32, 28672, 8192, 0, 0, T), (4, 96, 28672, 8192, 0, 1, T), (4, 65, 28672, 8192, 0, 0, M_), (4, 64, 11008, 4096, 0, 0, M_),
    # many tokens on few channels: what the L2s fetch of the activations counts
    (4, 4096, 11008, 64, 0, 0, T), (4, 2048, 11008, 128, 8, 0, T), (4, 1024, 11008, 512, 0, 0, T), (4, 1024, 11008, 1024, 0, 1, T),
    (4, 1024, 11008, 1024, 8, 0, M_), (4, 4096, 4096, 256, 0, 1, T), (4, 4096, 4096, 256, 0, 0, M_), (4, 4096, 4096, 64, 0, 1, M_),
    (4, 2048, 2048, 512, 8, 1, M_), (8, 2048, 11008, 512, 0, 1, T), (8, 2048, 11008, 512, 0, 0, M_), (8, 2048, 11008, 64, 0, 1, M_),
    # E4M3 weights: near 256 tiles, weights beyond what HBM hides; the streaming kernel's corners
    (8, 96, 12288, 16384, 0, 0, T), (8, 64, 12288, 16384, 0, 1, M_), (8, 256, 28672, 8192, 0, 0, T), (8, 32, 8192, 28672, 0, 0, T),
    (8, 24, 6144, 24576, 0, 1, T), (8, 9, 9216, 8192, 0, 0, S), (8, 12, 9216, 8192, 0, 0, M_), (8, 17, 2048, 4096, 0, 0, S),
    (8, 17, 2048, 4096, 8, 0, M_), (8, 24, 4096, 4096, 0, 1, S), (8, 24, 4096, 4096, 0, 0, M_), (8, 24, 3072, 3072, 0, 1, M_),
    (8, 16, 4096, 4096, 0, 0, D), (4, 16, 28672, 4096, 0, 0, D), (4, 16, 4096, 12288, 0, 0, D)])
def test_which_kernel_serves_a_gemm(lib, wbits, M, K, N, r, accum, form):
    """The choice is host logic; each of these is where one kernel measured faster than the other by 3 % or more
    (the figures stand at the rule), or a plain member of a form's range.  With 17 to 64 tokens, and where very many tokens meet few
    channels, "the other" is the tiled kernel with two by two waves a tile, against which the line was drawn: with four wave groups it is
    ahead of the form for a few dozen tokens at some of these points, by less than 10 %."""
    assert zqfp.probe_gemm_form(M, K, N, 128, wbits, r, accum) == form


def test_gemm_form_query_refuses_what_the_gemm_refuses(lib):
    for args in ((0, 4096, 4096), (1, 4000, 4096), (1, 4096, 0), (1, 4096, 4096, 96), (1, 4096, 4096, 64, 8), (1, 4096, 4096, 128, 5),
                 (1, 4096, 4096, 128, 4, 65)):
        with pytest.raises(zqfp.ZqfpError) as e:
            zqfp.probe_gemm_form(*args)
        assert e.value.code == -2
    with pytest.raises(zqfp.ZqfpError) as e:
        zqfp.probe_gemm_form(1, 4096, 4096, accum=2)
    assert e.value.code == -4


def test_extension_module_is_named_after_what_it_was_built_for():
    """It speaks the interpreter's and torch's binary interfaces; one built for others must not be loaded."""
    import sysconfig

    import torch
    name = os.path.basename(zqfp.BINDING_PATH)
    assert torch.__version__ in name and name.endswith(sysconfig.get_config_var("EXT_SUFFIX"))


def test_library_loads_without_the_extension_module(lib, monkeypatch, tmp_path):
    """Every call has its Python code; only the library itself is needed."""
    monkeypatch.setattr(zqfp, "_lib", None)
    monkeypatch.setattr(zqfp, "_native", None)
    monkeypatch.setattr(zqfp, "BINDING_PATH", str(tmp_path / "absent.so"))
    assert zqfp.lib().zqfp_version() >= 100
    for call, count in ((zqfp._native.quantize, 7), (zqfp._native.gemm, 10), (zqfp._native.linear, 8)):
        assert call(*[None] * count) is None


def test_library_is_built_by_hipcc_alone(monkeypatch, tmp_path):
    """The C library needs no C++ compiler of its own, no torch and no Python headers; those are the extension module's."""
    from paper_2307_09782_amd import build
    commands = []
    monkeypatch.setattr(build, "_run", lambda cmd: commands.append(cmd) or "")
    monkeypatch.setattr(build, "OBJDIR", str(tmp_path))
    monkeypatch.setattr(build.check_lds_waits, "check_text", lambda *a: None)
    for src in build.HAND_WAIT_SOURCES:
        (tmp_path / (src[:-4] + "-hip-amdgcn-amd-amdhsa-gfx950.s")).write_text("")
    build.build_lib()
    assert len(commands) == len(build.sources()) + 1
    assert {cmd[0] for cmd in commands} == {build.HIPCC}


B_, O, A = zqfp.LEFT_BLOCKS, zqfp.LEFT_ONE, zqfp.LEFT_APART


@pytest.mark.parametrize("kind,M,K,r,form", [
    # rows beyond 8192 elements behind a producer: the second block of ranks is a second round of workgroups from 129 tokens on
    (2, 128, 13440, 16, B_), (2, 223, 13440, 16, O), (2, 168, 12288, 16, O), (1, 187, 9728, 15, O), (3, 220, 8832, 12, O), (4, 256, 11008, 9, O),
    (1, 512, 4096, 16, B_), (1, 513, 4096, 16, O), (0, 512, 11008, 16, B_),
    # the plain quantizer with ranks one at a time: 768 tokens in one round, apart behind that and for long rows
    (0, 640, 128, 9, B_), (0, 768, 2048, 12, B_), (0, 769, 2048, 12, A), (0, 513, 20224, 9, A), (0, 720, 11008, 15, A),
    # sixteen ranks in one load: apart pays off later, behind a normalisation the later the longer the row
    (3, 1024, 8192, 16, O), (0, 1024, 8192, 16, O), (0, 800, 14336, 16, O), (0, 1300, 8192, 16, A), (3, 800, 8192, 15, A), (2, 1400, 8192, 16, O), (2, 1600, 2048, 16, O),
    (1, 2048, 2048, 16, A), (2, 1400, 9088, 16, O), (2, 1800, 9088, 16, A), (1, 1400, 8192, 15, A), (4, 4096, 4096, 16, O)])
def test_how_the_left_factor_is_formed(lib, kind, M, K, r, form):
    """Host logic; each of these is where one form measured faster than another by 4 % or more, or a neighbour across such a line."""
    assert zqfp.probe_left_form(M, K, r, kind) == form


def test_left_form_with_a_row_that_cannot_be_formed_twice(lib):
    """H over an operand: more than one workgroup per token would read what another has written."""
    for kind in (1, 2, 4):
        for M in (1, 16, 300, 5000):
            for r in range(9, 65):
                assert zqfp.probe_left_form(M, 4096, r, kind, in_place=True) != zqfp.LEFT_BLOCKS
    for args in ((0, 4096, 8), (1, 4100, 8), (1, 4096, 0), (1, 4096, 65), (1, 4096, 8, 5), (1, 32896, 8, 1)):
        with pytest.raises(zqfp.ZqfpError):
            zqfp.probe_left_form(*args)


def test_tile_plan_query_and_hook(lib):
    """The plan of a problem, what the hook puts in its place (the E4M3 form's two kernels of one shape included), and what both refuse."""
    try:
        for occ in (2, 3):
            zqfp.probe_force_tile_plan(64, 128, 1, 1, occ)
            assert zqfp.probe_tile_plan(1000, 4096, 11008, wbits=8) == (64, 128, 1, occ, 1, 32)
        zqfp.probe_force_tile_plan(64, 96, 3, 4)
        assert zqfp.probe_tile_plan(90, 2688, 210)[:3] == (64, 96, 4) and zqfp.probe_tile_plan(90, 2688, 210)[4:] == (3, 7)
        assert zqfp.probe_tile_plan(90, 2688, 210, have_workspace=False)[4:] == (1, 21)
        for args in ((64, 64, 1, 1), (64, 128, 1, 3), (128, 128, 1, 2), (64, 128, 65, 1), (64, 128, 1, 1, 4), (64, 128, 1, 2, 2), (128, 128, 1, 1, 2)):
            with pytest.raises(zqfp.ZqfpError):
                zqfp.probe_force_tile_plan(*args)
    finally:
        zqfp.probe_force_tile_plan()
    assert zqfp.probe_tile_plan(257, 11008, 4096)[2] == 4
    for args in ((0, 4096, 64), (64, 4100, 64), (64, 4096, 0), (64, 4096, 64, 5), (64, 4096, 64, 4, 2)):
        with pytest.raises(zqfp.ZqfpError):
            zqfp.probe_tile_plan(*args)
