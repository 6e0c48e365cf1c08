"""Host-side checks of the C-ABI library: it loads, exports every symbol the header declares, its
size helpers agree with the format description, and argument errors are reported without
launching anything (these calls return before the first HIP call, so they run without a GPU)."""
import ctypes
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    from paper_2603_27914_amd import binding, build

    if not os.path.exists(binding.LIB_PATH):
        build.build_lib()
    return binding.lib()


def declared_functions():
    names = set()
    for header in ("itq3s.h", "itq3s_bench.h"):  # the product interface and the measurement aids
        text = open(os.path.join(ROOT, "include", header)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(itq3s_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_product_header_keeps_its_contract():
    """Nothing that waits for the device is declared in the product header."""
    text = open(os.path.join(ROOT, "include", "itq3s.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    assert "_timed" not in text and "read_probe" not in text and "kernel_ms" not in text


def test_library_exports_every_declared_symbol(L):
    from paper_2603_27914_amd import binding

    names = declared_functions()
    assert len(names) >= 8
    for n in names:
        assert hasattr(L, n), n
    assert sorted(binding.EXPORTS) == names
    for n in names:  # the Python binding carries the same names
        if n != "itq3s_strerror":
            assert hasattr(binding, n), n


def test_size_helpers(L):
    assert L.itq3s_codes_bytes(16, 256) == 1536 and L.itq3s_scales_bytes(16, 256) == 64
    assert L.itq3s_codes_bytes(17, 512) == 2 * 2 * 1536
    assert L.itq3s_codes_bytes(2048, 2048) + L.itq3s_scales_bytes(2048, 2048) == 2048 * 8 * 100
    assert L.itq3s_codes_bytes(16, 255) == 0 and L.itq3s_scales_bytes(0, 256) == 0
    # the 70B-shaped stream: 267,386,880 blocks of 100 bytes
    from paper_2603_27914_amd import synth

    total = sum(c * (L.itq3s_codes_bytes(n, k) + L.itq3s_scales_bytes(n, k)) for _, n, k, c in synth.LLAMA70B_LAYER) * 80
    assert total == 26_738_688_000
    assert L.itq3s_matmul_workspace_bytes(1, 4096, 4096) == 256 and L.itq3s_matmul_workspace_bytes(4, 4096, 28672) == 256
    assert L.itq3s_matmul_workspace_bytes(8, 4096, 4096) >= 8 * 4096 * 2 + 8 * 16 * 8
    assert L.itq3s_matmul_workspace_bytes(512, 4096, 4096) >= 512 * 4096 * 2
    assert L.itq3s_version() >= 100


def test_argument_errors_return_before_any_launch(L):
    buf = (ctypes.c_uint8 * 4096)()
    p = ctypes.cast(buf, ctypes.c_void_p)
    addr = (p.value + 255) & ~255
    ok = ctypes.c_void_p(addr)
    odd = ctypes.c_void_p(addr + 2)
    assert L.itq3s_quantize(None, 16, 256, 256, ok, ok, None, None) == -1
    assert L.itq3s_quantize(ok, 16, 250, 256, ok, ok, None, None) == -2
    assert L.itq3s_quantize(ok, 0, 256, 256, ok, ok, None, None) == -2
    assert L.itq3s_quantize(ok, 16, 256, 128, ok, ok, None, None) == -2
    assert L.itq3s_quantize(odd, 16, 256, 256, ok, ok, None, None) == -3
    assert L.itq3s_quantize(ok, 16, 256, 258, ok, ok, None, None) == -3
    assert L.itq3s_dequantize(ok, ok, 16, 256, ok, 7, 256, None, None) == -4
    assert L.itq3s_dequantize(ok, None, 16, 256, ok, 0, 256, None, None) == -1
    assert L.itq3s_matmul(ok, ok, 16, 256, ok, 1, 256, ok, 0, 16, None, 0, None, None) == -5
    assert L.itq3s_matmul(ok, ok, 16, 256, ok, 1, 256, ok, 0, 16, ok, 8, None, None) == -5
    assert L.itq3s_matmul(ok, ok, 16, 256, ok, 8, 256, ok, 0, 16, ok, 1024, None, None) == -5
    assert L.itq3s_matmul(ok, ok, 16, 1 << 29, ok, 1, 1 << 29, ok, 0, 16, ok, 1 << 20, None, None) == -2
    assert L.itq3s_matmul(ok, ok, 16, 256, ok, 1, 256, ok, 0, 8, ok, 1 << 20, None, None) == -2
    assert L.itq3s_matmul(ok, ok, 16, 256, ok, 1, 250, ok, 0, 16, ok, 1 << 20, None, None) == -2
    assert L.itq3s_matmul(ok, ok, 16, 256, ok, 1, 260, ok, 0, 16, ok, 1 << 20, None, None) == -3
    assert L.itq3s_matmul(ok, ok, 16, 256, ok, 1, 256, ok, 3, 16, ok, 1 << 20, None, None) == -4
    for code in range(0, -7, -1):
        assert len(L.itq3s_strerror(code)) > 0
    assert L.itq3s_strerror(-99) == b"unknown status"


def test_binding_refuses_cpu_tensors():
    import torch

    from paper_2603_27914_amd import binding

    with pytest.raises(binding.Itq3sError):
        binding.itq3s_quantize(torch.zeros(16, 256))


def test_binding_imports_on_a_torch_without_device_support():
    """Such a torch has no stream accessors; only the calls that need a device fail there."""
    code = (
        "import torch\n"
        "for name in ('_cuda_getCurrentRawStream', '_cuda_getDevice'):\n"
        "    if hasattr(torch._C, name): delattr(torch._C, name)\n"
        "from paper_2603_27914_amd import binding\n"
        "assert binding.itq3s_codes_bytes(16, 256) == 1536\n"
        "try: binding.itq3s_quantize(torch.zeros(16, 256))\n"
        "except binding.Itq3sError: pass\n"
        "else: raise AssertionError('a CPU tensor was accepted')\n"
    )
    subprocess.run([sys.executable, "-c", code], check=True, cwd=ROOT)


def test_binding_checks_packed_tensors_against_the_shape():
    """The C ABI takes pointers and trusts N and K; the binding refuses tensors that do not hold
    W[N, K] before anything is launched (a kernel reading past them would fault the device)."""
    import torch

    from paper_2603_27914_amd import binding

    N, K = 40, 512
    cw, sw = binding.itq3s_codes_bytes(N, K) // 4, binding.itq3s_scales_bytes(N, K) // 4
    codes, scales = torch.zeros(cw, dtype=torch.int32), torch.zeros(sw, dtype=torch.int32)
    binding._need_packed(codes, scales, N, K)  # fits
    binding._need_packed(codes, scales, 33, K)  # same number of row tiles
    for bad_args, what in [
        ((codes, scales, 64, K), "holds"),                      # more rows than stored
        ((codes, scales, N, 1024), "holds"),                    # longer rows than stored
        ((codes[:-1], scales, N, K), "holds"),                  # a tensor cut short
        ((codes, scales[: sw // 2], N, K), "holds"),
        ((codes, scales, N, 500), "bad shape"),                 # K not a multiple of 256
        ((codes, scales, 0, K), "bad shape"),
        ((codes.to(torch.int64), scales, N, K), "int32"),       # wrong element type
        ((codes, scales.float(), N, K), "int32"),
        ((torch.zeros(2 * cw, dtype=torch.int32)[::2], scales, N, K), "contiguous"),  # a strided view
    ]:
        with pytest.raises(binding.Itq3sError, match=what):
            binding._need_packed(*bad_args)
    with pytest.raises(binding.Itq3sError, match="status_flags"):
        binding._need_flags(torch.zeros(0, dtype=torch.int32))
    with pytest.raises(binding.Itq3sError, match="status_flags"):
        binding._need_flags(torch.zeros(1, dtype=torch.float32))
    binding._need_flags(None)
    binding._need_flags(torch.zeros(1, dtype=torch.int32))


def test_dequantize_stores_promise_no_more_alignment_than_the_header():
    """The output's rows start at multiples of four elements: 16 bytes in fp32, eight in fp16.  The fp16 kernels
    store four 32-bit words at once, which must not claim 16-byte alignment (read from the compiler's
    intermediate code: the hardware accepts the access either way)."""
    from paper_2603_27914_amd import build

    src = os.path.join(build.CSRC, "itq3s_dequantize.hip")
    cmd = ["hipcc", *build.flags(src), "--cuda-device-only", "-S", "-emit-llvm", src, "-o", "-"]
    ir = subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True).stdout
    stores = re.findall(r"store <4 x (i32|float)> .*, align (\d+),.* !nontemporal", ir)
    assert {t for t, _ in stores} == {"i32", "float"}
    assert {a for t, a in stores if t == "i32"} == {"8"} and {a for t, a in stores if t == "float"} == {"16"}


def test_settings_kept_per_device_are_made_on_every_device(tmp_path):
    """A kernel's limit of dynamic LDS belongs to one device: each device that the process runs on gets it
    once, a failure is not remembered, devices beyond the remembered ones get it on every call."""
    main = tmp_path / "once.cpp"
    main.write_text(
        '#include "itq3s_once.h"\n'
        "#include <cstdio>\n"
        "int main() {\n"
        "    static itq3s::DeviceOnce once;\n"
        "    const int devices[] = {0, 0, 1, 0, 1, 63, 63, 64, 64, 2, 2, 2};\n"
        "    int calls = 0;\n"
        "    for (int d : devices) {\n"
        "        bool called = false;\n"
        "        const bool ok = once(d, [&] { called = true; return d != 2 || ++calls > 1; });\n"
        '        std::printf("%d%d ", (int)called, (int)ok);\n'
        "    }\n"
        "}\n"
    )
    from paper_2603_27914_amd import build

    exe = tmp_path / "once"
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(main), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, stdout=subprocess.PIPE, text=True).stdout.split()
    #                    0     0     1     0     1     63    63    64    64    2 (fails) 2     2
    assert out == ["11", "01", "11", "01", "01", "11", "01", "11", "11", "10", "11", "01"]
    for name in os.listdir(build.CSRC):  # ... and nothing raises the limit in another way
        if name.endswith((".hip", ".h")) and name != "itq3s_kernels.h":
            assert "hipFuncSetAttribute" not in open(os.path.join(build.CSRC, name)).read(), name


@pytest.mark.parametrize("source", ["gemv", "rows", "rotate", "gemm", "mx", "gemm_ws", "dequantize", "quantize"])
def test_kernels_keep_their_registers(source):
    """No kernel of the path parks registers in scratch memory (a spill in one of the many instantiations of a
    kernel costs time and nothing else, so no other test sees it)."""
    from paper_2603_27914_amd import build

    src = os.path.join(build.CSRC, "itq3s_%s.hip" % source)
    cmd = ["hipcc", *build.flags(src), "--cuda-device-only", "-S", src, "-o", "-"]
    asm = subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True).stdout
    kernels = re.findall(r"\.amdhsa_kernel (\S+).*?\.amdhsa_private_segment_fixed_size (\d+)", asm, flags=re.S)
    assert kernels and [k for k in kernels if k[1] != "0"] == []
    # the copies written in assembly set m0, which cannot be named as clobbered: where there are any, nothing else uses it
    written, other = [], []
    for block in re.split(r"(;;?#ASMSTART.*?;;?#ASMEND)", asm, flags=re.S):
        (written if block.lstrip(";").startswith("#ASMSTART") else other).append(block)
    assert not any(re.search(r"\bm0\b", b) for b in written) or not any(re.search(r"^\s+\w.*\bm0\b", b, flags=re.M) for b in other)
    assert source != "gemm" or any(re.search(r"\bm0\b", b) for b in written)


# us a call (weights cycled through memory): M, N, K, the tiled kernel (17 rows: two passes of the kernel for 16
# rows) before the many-row kernel was there, the same now, the many-row kernel
ROUTES = [
    (3200, 1000, 256, 22.4, 17.1, 25.2), (300, 11008, 256, 22.1, 17.1, 23.5), (65, 28672, 256, 18.4, 16.1, 20.2), (112, 28672, 256, 21.0, 16.7, 23.4),
    (33, 57344, 256, 17.1, 16.5, 19.6), (64, 128256, 256, 24.0, 22.0, 41.7), (64, 57344, 512, 22.6, 20.9, 23.9), (33, 128256, 512, 28.5, 27.6, 36.4),
    (56, 128256, 1024, 43.4, 41.5, 48.5), (4096, 600, 2048, 40.9, 35.8, 43.6), (3200, 1000, 2048, 40.2, 35.8, 50.9), (2048, 1500, 2048, 38.4, 34.6, 43.5),
    (1500, 1000, 4096, 39.5, 35.9, 41.2), (2048, 1000, 4096, 44.6, 40.5, 52.1), (2048, 1500, 4096, 55.8, 51.8, 71.8), (1500, 2048, 4096, 53.5, 50.1, 58.7),
    (1800, 600, 8192, 61.8, 52.6, 68.8), (1800, 1000, 8192, 71.3, 59.8, 83.8), (17, 16, 28672, 27.8, 26.7, 30.5), (17, 300, 28672, 32.4, 31.5, 33.8),
    (33, 11008, 256, 16.1, 15.4, 8.4), (64, 20000, 256, 18.2, 15.8, 12.1), (384, 3072, 256, 21.4, 16.4, 12.0), (1024, 2048, 512, 25.0, 20.0, 16.0),
    (64, 28672, 1024, 27.3, 25.6, 16.1), (512, 4096, 1024, 31.5, 26.6, 17.1), (1024, 2048, 2048, 36.5, 34.0, 24.4), (1024, 1000, 4096, 36.6, 33.5, 24.1),
    (1024, 2048, 4096, 41.4, 38.6, 36.4), (300, 11008, 4096, 67.8, 62.4, 52.1), (64, 28672, 8192, 78.5, 80.3, 52.2), (64, 11008, 14336, 67.2, 63.0, 39.5),
    (24, 4096, 28672, 44.7, 44.2, 35.4), (512, 600, 28672, 79.5, 73.5, 56.8), (1800, 16, 8192, 42.3, 36.0, 27.4), (6000, 128, 2048, 41.0, 34.5, 23.4),
    (1200, 2048, 2048, 37.0, 34.3, 31.9), (1800, 1000, 2048, 37.2, 33.6, 30.8), (4096, 300, 2048, 39.7, 33.8, 33.2), (2600, 600, 4096, 46.3, 41.6, 47.5),
]


def test_no_call_goes_to_the_slower_kernel(tmp_path):
    """rows_path, which calls the many-row kernel may take: only where it beats what computed them before, and wherever it
    clearly does (sizes on both sides of each line of the rule, with the times that were measured; the tiled kernel had
    fp16 operands then.  Between it and the block-scaled kernels many_row_route decides, by times of its own)."""
    from paper_2603_27914_amd import build

    main = tmp_path / "rule.cpp"
    main.write_text(
        '#include "itq3s_rows_rule.h"\n#include <cstdio>\n'
        "int main() { long long M, N, K;\n"
        '    while (std::scanf("%lld %lld %lld", &M, &N, &K) == 3) std::printf("%d ", (int)itq3s::rows_path(M, N, K)); }\n'
    )
    exe = tmp_path / "rule"
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(main), "-o", str(exe)], check=True)
    sizes = "".join("%d %d %d\n" % r[:3] for r in ROUTES)
    taken = [int(v) for v in subprocess.run([str(exe)], input=sizes, check=True, stdout=subprocess.PIPE, text=True).stdout.split()]
    for (M, N, K, before, other, rows), many in zip(ROUTES, taken):
        chosen = rows if many else other
        assert chosen <= before * 1.03 and chosen <= 1.05 * min(rows, other), (M, N, K, many)
