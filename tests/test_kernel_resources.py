"""No kernel that runs in a workload's step may use scratch memory (a spill in one kernel slowed every other kernel of
the step when it was measured).  Compiles the device code once with hipcc's resource-usage remarks and checks every
kernel; runs without a GPU."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1811_03115_amd import build

# Instantiations that exist in the library but that no dispatch rule reaches with the shapes of any workload here
# (the widest skinny-GEMM forms with a LayerNorm epilogue or two column tiles per wave), and the opt-in decoder stack
# kernel, whose 36-byte frame holds no spilled register (no scratch instruction in its code).
ALLOWED = [
    r"skinny_gemm_kernel<1, 2, false, (false|true), 8, 16, [01], (false|true)>",
    r"skinny_gemm_kernel<1, 1, false, false, 8, 16, 1, (false|true)>",
    r"decoder_stack_kernel<\d+>",
]
# kernels that must be there and scratch-free, besides those that the traces of the timed cases name (traced()): a choice of the latter, and those that other
# widths, depths and row counts run in their place
REQUIRED = [
    "row_gemm_kernel<8, 4, 1, 1, true, 0>", "row_gemm_kernel<8, 4, 1, 1, true, 2>", "row_gemm_kernel<8, 4, 1, 1, false, 1>",
    "row_gemm_kernel<8, 4, 1, 1, false, 2>", "row_gemm_kernel<8, 4, 1, 1, false, 3>", "row_gemm_kernel<8, 4, 2, 4, false, 0>",
    "row_gemm_kernel<8, 4, 4, 4, false, 2>", "row_gemm_kernel<4, 4, 1, 1, true, 0>", "row_gemm_kernel<4, 4, 1, 1, true, 2>",
    "row_gemm_kernel<4, 4, 1, 1, false, 1>", "row_gemm_kernel<8, 8, 1, 1, false, 1>",
    "ln_row_kernel<1024, 4>", "ln_row_kernel<1024, 0>", "ln_row_kernel<512, 0>",
    "attention_mfma_kernel<false, false, 8>", "attention_mfma_kernel<false, false, 4>", "attention_mfma_kernel<false, false, 0>",
    "attention_mfma_kernel<false, true, -1>", "attention_mfma_kernel<true, false, -1>", "attention_mfma_slots_kernel<false, true, 0>",
    "attention_mfma_slots_kernel<false, true, -1>",
    "skinny_gemm_kernel<1, 2, false, false, 4, 8, 2, true>", "skinny_gemm_kernel<1, 1, false, false, 8, 8, 0, false>",
    "stream_gemm_kernel<16, true>", "stream_vocab_kernel<4, 1, 2, false>", "stream_vocab_kernel<4, 1, 1, false>",
    "gemm_ldsx_kernel<8, 4, 64, true, false, false, false>", "gemm_ldsx_kernel<7, 4, 64, false, false, false, false>",
    "gemm_ldsx_kernel<4, 2, 128, false, false, false, false>",
    "small_decode_kernel<1>", "small_encode_kernel", "small_prime_kernel", "accept_embed_kernel", "encode_init_kernel", "decode_init_kernel", "fetch_kernel",
    "skinny_gemm_kernel<1, 1, false, false, 8, 16, 0, false>", "skinny_gemm_kernel<1, 1, false, false, 4, 8, 0, false>",
    "gemm_ldsx_kernel<1, 1, 256, false, false, true, false>", "gemm_ldsx_kernel<1, 1, 256, false, true, false, false>", "gemm_ldsx_kernel<1, 1, 256, false, false, false, true>",
    "layernorm_kernel<unsigned short, 4>",
    "layers_kernel<2048, false>", "layers_kernel<2048, true>", "wide_layers_kernel", "tall_layers_kernel<2>", "tall_layers_kernel<3>", "tall_layers_kernel<4>", "topn_rank_kernel",
]


def traced():
    """The library's kernels in profiles/case_kernel_traces.txt, with their template arguments."""
    with open(os.path.join(os.path.dirname(__file__), "..", "profiles", "case_kernel_traces.txt")) as f:
        names = re.findall(r"^  (?:void )?(\w+(?:<[^>]*>)?)\(", f.read(), re.M)
    assert len(names) > 100
    return sorted(set(names))


def test_no_step_kernel_uses_scratch(tmp_path):
    hipcc = build.hipcc()
    if shutil.which(hipcc) is None and not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [hipcc] + flags + ["--cuda-device-only", "-c", build.SOURCES[0], "-o", str(tmp_path / "dev.o"),
                             "-Rpass-analysis=kernel-resource-usage"]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-2000:]
    names, scratch = [], {}
    cur = None
    for line in res.stdout.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = m.group(1)
            names.append(cur)
            continue
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m and cur is not None:
            scratch[cur] = int(m.group(1))
    assert len(names) > 100, "resource remarks missing"
    dem = subprocess.run(["c++filt"] + names, stdout=subprocess.PIPE, text=True).stdout.splitlines()
    by_name = dict(zip(dem, (scratch[n] for n in names)))
    offenders = [f"{n}: {s} bytes" for n, s in by_name.items() if s > 0 and not any(re.search(a, n) for a in ALLOWED)]
    assert not offenders, "kernels with scratch memory:\n" + "\n".join(offenders)
    for req in REQUIRED + traced():
        hits = [n for n in by_name if re.search(r"(^|\W)" + re.escape(req) + r"(\W|$)", n)]
        assert hits, f"kernel {req} not found"
        assert all(by_name[n] == 0 for n in hits), f"{req} uses scratch"


def waves_of(tmp_path, instantiations):
    """[(mangled name, waves per SIMD that the registers leave room for)] of explicit instantiations of kernels."""
    hipcc = build.hipcc()
    if shutil.which(hipcc) is None and not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    src = tmp_path / "kernels.hip"
    src.write_text(f'#include "{os.path.dirname(build.SOURCES[0])}/bpd_kernels.h"\n' + "".join(f"template __global__ void {i};\n" for i in instantiations))
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([hipcc] + flags + ["--cuda-device-only", "-c", str(src), "-o", str(tmp_path / "kernels.o"), "-Rpass-analysis=kernel-resource-usage"],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-2000:]
    return [(n, int(w)) for n, w in re.findall(r"Function Name: (\S+).*?Occupancy \[waves/SIMD\]: (\d+)", res.stdout, re.S)]


def tile_waves(tmp_path, tiles):
    """Those of gemm_ldsx_kernel<MT, NT, KC>, plain and with arg-max."""
    got = waves_of(tmp_path, [f"gemm_ldsx_kernel<{mt}, {nt}, {256 // nt}, {m}, false, false, false>(GemmP, Epi, unsigned long long*, float*, LnP, LiveP)"
                              for mt, nt in tiles for m in ("false", "true")])
    found = [(re.match(r"_Z\d+gemm_ldsx_kernelILi(\d)ELi(\d)ELi\d+ELb([01])E", n), w) for n, w in got]
    found = {(int(m[1]), int(m[2]), m[3] == "1"): w for m, w in found if m}
    assert len(found) == 2 * len(tiles)
    return found


def test_combine_waves(tmp_path):
    """Sixteen partial results per thread: 64 registers of values, and not as many again for where they go."""
    got = waves_of(tmp_path, [f"attention_combine_kernel<{act}, {dh}, 16>(AttnP)" for act, dh in (("bf16_t", 64), ("bf16_t", 16), ("float", 16))])
    got = [w for n, w in got if "attention_combine_kernel" in n]
    assert len(got) == 3 and min(got) >= 5, got


def test_workgroups_side_by_side(tmp_path):
    """The tile rule's count of workgroups per CU is what registers and LDS of the built kernels allow (four waves each); tiles of 256 columns: three up to 64 rows, four up to 32."""
    tiles = [(mt, nt) for nt in (1, 2, 4) for mt in (1, 2, 3, 4, 5, 7, 8) if nt > 1 or mt <= 3]
    src = tmp_path / "count.cpp"
    src.write_text(f'#include <cstdio>\n#include "{os.path.dirname(build.SOURCES[0])}/bpd_host_logic.h"\nint main() {{ for (int nt : {{1, 2, 4}}) for (int mt = 1; mt <= 8; ++mt) printf("%d %d %d\\n", mt, nt, ldsx_side_by_side(mt, nt)); }}\n')
    subprocess.run(["g++", "-std=c++17", str(src), "-o", str(tmp_path / "count")], check=True)
    count = {(mt, nt): n for mt, nt, n in (map(int, line.split()) for line in subprocess.run([str(tmp_path / "count")], stdout=subprocess.PIPE, text=True).stdout.splitlines())}
    waves = tile_waves(tmp_path, tiles)
    for (mt, nt, argmax), w in waves.items():
        deep = nt == 4 and mt >= 4
        lds = (3 if deep else 2) * ((16 * mt * (256 // nt // 8) + 255) // 256) * 4096
        if not argmax:
            assert count[mt, nt] == min(4, w, 160 * 1024 // lds), f"{16 * mt} x {64 * nt}: {w} waves per SIMD, {lds} bytes of LDS"
        if nt == 4:
            assert w == (4 if mt <= 2 else (3 if mt <= 4 else 2)), f"{16 * mt} x 256: {w} waves per SIMD"
