"""What the compiler made of load hints and registers, which results do not show: built for gfx950 from the kernels' header, no
device."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2104_06069_amd", "csrc")
PASS = """
#define PASS(KEEP) template __global__ void obk::k_ratios_pass<1, false, false, KEEP>( \\
    RatioArgs, float*, int64_t, int, LayerTab, const int*, const int*, const int*);
PASS(false)
PASS(true)
"""
HIST = """
#define HIST(K, LP, S) template __global__ void obk::k_ratios_apply_hist<K, LP, S, false>( \\
    RatioArgs, VfHist, VTerms, ApplyArgs, LayerSync, LayerTab);
HIST(false, false, 0) HIST(false, true, 0) HIST(true, false, 0) HIST(true, true, 0)
HIST(false, false, 6) HIST(false, true, 6) HIST(true, false, 6) HIST(true, true, 6)
"""
BIG = """
#define BIG(K) template __global__ void obk::k_ratios_big_hist<K>(RatioArgs, VfHist, VTerms, float*, const int*, int64_t, int, int, \\
                                                                  LayerTab, const int*);
BIG(false) BIG(true)
"""
WORKER = """
#define WORKER(K, GT, LDS) template __global__ void obk::k_momentum_z_sumsq<1, K, true, GT, true, false, LDS>( \
    GradSrc, const float*, PackedMom, float*, double*, int64_t, int, float, float, LayerTab, PackedErr, uint32_t*, OwnCopy, ChunkTicket);
WORKER(false, 0, false) WORKER(false, 1, false) WORKER(true, 1, false) WORKER(false, 1, true)
"""
RESIDENT = """
#define RESIDENT(K, LP) template __global__ void obk::k_ratios_apply_resident<8, K, LP>(RatioArgs, ApplyArgs, LayerSync, LayerTab);
RESIDENT(false, false) RESIDENT(false, true) RESIDENT(true, false) RESIDENT(true, true)
"""
TRAIL = """
#define TRAIL(K, LP) template __global__ void obk::k_ratios_trail<K, LP>(RatioArgs, VfHist, VTerms, ApplyArgs, RatioTrailTab, LayerTab);
TRAIL(false, false) TRAIL(false, true) TRAIL(true, false) TRAIL(true, true)
"""
LAMB = """
#define LAMB(GT, LP) template __global__ void obk::k_warmup_resident<8, 1, GT, LP>( \\
    GradSrc, float*, float*, float*, WarmSync, float, float, float, float, float, float, float, LayerTab, void*, int);
LAMB(0, false) LAMB(0, true) LAMB(1, false) LAMB(1, true)
"""


def assembly(tmp_path, kernels):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text('#include "ob_kernels.h"\nusing namespace obk;\n' + kernels)
    subprocess.run([hipcc, "-O3", "--offload-arch=gfx950", "--offload-device-only", "-S", "-std=c++17", "-ffp-contract=off",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", CSRC, str(src), "-o", str(asm)],
                   check=True, capture_output=True)
    return asm.read_text()


def test_second_reads_are_kept_only_where_asked_for(tmp_path):
    """The ratio pass loads m, v_frozen and v_fresh past the caches, or v_frozen through them: one hint less."""
    text, hints = assembly(tmp_path, PASS), []
    for keep in "01":
        body = re.search(r"^_ZN3obk13k_ratios_passILi1ELb0ELb0ELb%s\w*:[^\n]*$(.*?)s_endpgm" % keep, text, re.S | re.M).group(1)
        hints.append(len(re.findall(r"global_load_dwordx4 .* nt$", body, re.M)))
    assert hints == [3, 2], hints


def test_worker_s_sum_of_squares_goes_through_lds_only_where_asked_for(tmp_path):
    """k_momentum_z_sumsq: six doubles and the sign word's three steps by ds_bpermute, or none."""
    text = assembly(tmp_path, WORKER)
    for k, gt, lds in ((0, 0, 0), (0, 1, 0), (1, 1, 0), (0, 1, 1)):
        body = re.search(r"^_ZN3obk18k_momentum_z_sumsqILi1ELb%dELb1ELi%dELb1ELb0ELb%dE\w*:[^\n]*$(.*?)^\.Lfunc_end" % (k, gt, lds), text,
                         re.S | re.M).group(1)
        assert len(re.findall(r"^\s+ds_bpermute_b32", body, re.M)) == 15 * lds, (k, gt, lds)


def spills(tmp_path, name, kernels):
    """(scalar, vector) registers that each instantiation of the kernel spills at the occupancy that it is built for."""
    counts = re.findall(r"\.name:\s+_ZN3obk%d%s.*?\.sgpr_spill_count:\s+(\d+).*?\.vgpr_spill_count:\s+(\d+)" % (len(name), name),
                        assembly(tmp_path, kernels), re.S)
    return [(int(a), int(b)) for a, b in counts]


@pytest.mark.parametrize("name,kernels,n", [("k_ratios_apply_hist", HIST, 8), ("k_ratios_big_hist", BIG, 2), ("k_ratios_apply_resident", RESIDENT, 4),
                                            ("k_ratios_trail", TRAIL, 4), ("k_warmup_resident", LAMB, 4)])
def test_kernels_of_the_large_lists_keep_their_registers(tmp_path, name, kernels, n):
    """The kernels of the large lists (k_ratios_apply_hist without the rest tiles in its launch) have no spills."""
    assert spills(tmp_path, name, kernels) == [(0, 0)] * n


def test_rest_tiles_in_the_launch_spill_hardly_any_vector_registers(tmp_path):
    """With the rest tiles in its launch k_ratios_apply_hist spills scalar registers, into the lanes of one vector register (64), and in some of
    its forms one vector register."""
    counts = spills(tmp_path, "k_ratios_apply_hist", HIST.replace("S, false>", "S, true>"))
    assert len(counts) == 8 and all(a <= 64 and b <= 1 for a, b in counts), counts


@pytest.mark.parametrize("name,kernels,loads,stores,n", [("k_ratios_apply_hist", HIST, (18, 24), 16, 8), ("k_ratios_big_hist", BIG, (16,), 8, 2)])
def test_tiles_are_addressed_by_a_scalar_base(tmp_path, name, kernels, loads, stores, n):
    """Their 16-byte accesses take a scalar base and a 32-bit lane offset: 64-bit vector addresses cost an addition with carry before each load."""
    bodies = re.findall(r"^_ZN3obk%d%s\w*:[^\n]*$(.*?)^\.Lfunc_end" % (len(name), name), assembly(tmp_path, kernels), re.S | re.M)
    assert len(bodies) == n
    for body in bodies:
        by_scalar = [len(re.findall(p, body)) for p in (r"global_load_dwordx4 v\[\d+:\d+\], v\d+, s\[", r"global_store_dwordx4 v\d+, v\[\d+:\d+\], s\[")]
        assert by_scalar[0] in loads and by_scalar[1] == stores, by_scalar
        assert not re.findall(r"global_(?:load|store)_dwordx4 v\[\d+:\d+\], (?:v\[\d+:\d+\], )?off", body)
