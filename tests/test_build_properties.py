"""What the compiler made of the hot kernels (no GPU needed: hipcc cross-compiles gfx950): none of them may spill
registers to scratch memory, and each has to keep the occupancy its launch bounds were chosen for."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2205_09707_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# kernel (prefix of the mangled name's readable part) -> (source file, most vector registers, most LDS bytes)
KERNELS = {
    "scq_mfma_kernelILi2E": ("k_scq.hip", 128, 40 << 10),          # four waves per SIMD, four workgroups per CU
    "scq_mfma_kernelILi1E": ("k_scq.hip", 128, 40 << 10),
    "stage1_tail_kernelILi2ELb0E": ("k_scq.hip", 128, 64 << 10),   # 1024 threads: 128 registers at most
    "stage1_tail_kernelILi8ELb0E": ("k_scq.hip", 128, 64 << 10),
    "stage1_tail_kernelILi2ELb1E": ("k_scq.hip", 128, 64 << 10),   # ... also with the re-evaluations in double
    "stage1_tail_kernelILi8ELb1E": ("k_scq.hip", 128, 64 << 10),
    "stage1_parts_kernelILi1E": ("k_scq.hip", 128, 64 << 10),      # the survivors' workgroup has 1024 threads
    "stage1_parts_kernelILi2E": ("k_scq.hip", 128, 64 << 10),
    "stage1_parts_kernelILi4E": ("k_scq.hip", 128, 64 << 10),
    "stage1_parts_kernelILi8E": ("k_scq.hip", 128, 64 << 10),
    "scq16_kernelILi2ELb1E": ("k_scq16.hip", 256, 40 << 10),   # two waves per SIMD, two to four workgroups per CU
    "scq16_kernelILi2ELb0E": ("k_scq16.hip", 256, 32 << 10),   # without group maxima: the two operand buffers and nothing else
    # a wave per 2048 passages, 256 threads: what the workgroups per compute unit that its launch bounds name can have
    "s2_invert_kernelILi11EjLb0ELb0ELb0E": ("k_stage2.hip", 128, 40 << 10),   # 32-bit sets: four
    "s2_invert_kernelILi11EjLb1ELb0ELb0E": ("k_stage2.hip", 128, 40 << 10),
    "s2_invert_kernelILi13EjLb0ELb0ELb0E": ("k_stage2.hip", 128, 40 << 10),
    "s2_invert_kernelILi13EjLb1ELb0ELb0E": ("k_stage2.hip", 128, 40 << 10),
    "s2_invert_kernelILi11EyLb0ELb0ELb0E": ("k_stage2.hip", 128, 40 << 10),   # 64-bit sets: four
    "s2_invert_kernelILi13EyLb0ELb0ELb0E": ("k_stage2.hip", 128, 40 << 10),
    "s2_invert_kernelILi11EyLb0ELb1ELb0E": ("k_stage2.hip", 128, 40 << 10),   # ... launched alone
    "s2_invert_kernelILi13EyLb0ELb1ELb0E": ("k_stage2.hip", 128, 40 << 10),
    "s2_invert_kernelILi11EyLb0ELb0ELb1E": ("k_stage2.hip", 168, 53 << 10),   # ... with 36 planes per wave: three
    "s2_invert_kernelILi11EyLb0ELb1ELb1E": ("k_stage2.hip", 168, 53 << 10),
    "s2_candidates_kernel": ("k_stage2.hip", 64, 8 << 10),
    "s2_union_wide_kernel": ("k_stage2.hip", 128, 80 << 10),       # two workgroups of 1024 threads per CU
    "s2_stream_kernel": ("k_stage2.hip", 128, 40 << 10),
    "ci_few_kernelILb0E": ("k_ci.hip", 64, 8 << 10),               # eight waves per SIMD
    "ci_list_kernelILb0E": ("k_ci.hip", 96, 8 << 10),              # five waves per SIMD; wave-private LDS areas
    "decompress_maxsim_kernelILi2ELb0ELb0ELb0E": ("k_stage4.hip", 128, 32 << 10),   # four waves per SIMD (query operands in LDS)
    "decompress_maxsim_kernelILi1ELb0ELb0ELb0E": ("k_stage4.hip", 128, 32 << 10),
    "decompress_maxsim_kernelILi2ELb0ELb0ELb1E": ("k_stage4.hip", 128, 32 << 10),   # ... with 64-bit offsets of rows
    "decompress_maxsim_kernelILi2ELb0ELb1ELb0E": ("k_stage4.hip", 128, 32 << 10),   # ... with unit-length reconstruction
    "cut_maxsim_kernelILi2ELb0ELb0E": ("k_stage4.hip", 128, 32 << 10),   # a workgroup per key: four waves per SIMD
    "cut_maxsim_kernelILi1ELb0ELb0E": ("k_stage4.hip", 128, 32 << 10),
    "cut_maxsim_kernelILi2ELb1ELb0E": ("k_stage4.hip", 128, 32 << 10),   # ... with unit-length reconstruction
    "cut_maxsim_kernelILi1ELb1ELb0E": ("k_stage4.hip", 128, 32 << 10),
    "cut_maxsim_kernelILi2ELb0ELb1E": ("k_stage4.hip", 128, 32 << 10),   # ... with 64-bit offsets of rows
    "cut_maxsim_kernelILi1ELb0ELb1E": ("k_stage4.hip", 128, 32 << 10),
    "cut_maxsim_kernelILi2ELb1ELb1E": ("k_stage4.hip", 128, 32 << 10),
    "cut_maxsim_kernelILi1ELb1ELb1E": ("k_stage4.hip", 128, 32 << 10),
    # three waves per SIMD, three workgroups per CU (the pruning instances add 8 KB of dynamic LDS)
    "maxsim_list_kernelILi2ELb1ELb0ELb0E": ("k_stage4.hip", 168, 45 << 10),
    "maxsim_list_kernelILi1ELb1ELb0ELb0E": ("k_stage4.hip", 168, 45 << 10),
    "maxsim_list_kernelILi2ELb0ELb0ELb0E": ("k_stage4.hip", 168, 53 << 10),
    "maxsim_list_kernelILi1ELb0ELb1ELb0E": ("k_stage4.hip", 168, 53 << 10),
    # four waves per SIMD, four workgroups per CU with the 8 KB of dynamic LDS
    "van_coarse_kernelILi2E": ("k_stage4.hip", 128, 32 << 10),
    "van_coarse_kernelILi1E": ("k_stage4.hip", 128, 32 << 10),
    "van_bounds_kernel": ("k_stage4.hip", 64, 1 << 10),
    "van_band_kernel": ("k_stage4.hip", 64, 1 << 10),
    "decompress_dump_kernelILi2E": ("k_stage4.hip", 64, 8 << 10),        # eight workgroups of 256 threads per CU
    "decompress_dump_kernelILi1E": ("k_stage4.hip", 64, 16 << 10),
    "passage_offsets_kernel": ("k_stage4.hip", 64, 1 << 10),
    "van_codes_kernel": ("k_vanilla.hip", 64, 1 << 10),
    "van_union_kernel": ("k_vanilla.hip", 64, 8 << 10),
    "asg_screen_kernel": ("k_assign.hip", 256, 20 << 10),          # two waves per SIMD: 128 registers of operands, 64 of results
    "asg_pick_kernel": ("k_assign.hip", 96, 32 << 10),             # five waves per SIMD, five workgroups per CU
    "sel_pick_kernel": ("k_select.hip", 64, 80 << 10),             # 1024 threads, two workgroups per CU
    "sel2_finish_kernel": ("k_select.hip", 64, 80 << 10),
    "sel_sort_kernelILi512E": ("k_select.hip", 64, 0),             # dynamic LDS only
    "sel2_filter_kernel": ("k_select.hip", 64, 8 << 10),
    "sel2_bins_kernel": ("k_select.hip", 80, 16 << 10),            # six waves per SIMD
    "sel2_cut_kernelILi1E": ("k_select.hip", 64, 80 << 10),        # 1024 threads, two workgroups per CU
    "sel2_cut_kernelILi2E": ("k_select.hip", 64, 80 << 10),
    "bitmap_to_list_kernel": ("k_util.hip", 64, 1 << 10),          # 1024 threads, two workgroups per CU
    "encode_residuals_kernelILi2E": ("k_build.hip", 64, 0),
    "ivb_rank_kernel": ("k_build.hip", 64, 0),
    "ivb_sort_short_kernel": ("k_build.hip", 64, 0),             # up to 32 entries per lane in registers: eight waves per SIMD
    "ivb_sort_long_kernel": ("k_build.hip", 128, 130 << 10),     # a bitmap of 2^20 passage ids: one workgroup (16 waves) per CU
}


def _assembly(src, out):
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fno-gpu-rdc", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "--cuda-device-only", "-S",
           os.path.join(CSRC, src), "-o", out]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return open(out).read()


def _metadata(text):
    """name -> dict of the integer fields of each kernel's metadata record"""
    out = {}
    for rec in text.split("  - .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", rec).group(1)
        f = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\n", rec)}
        f["agpr_count"] = int(rec.split("\n", 1)[0])
        out[name] = f
    return out


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not installed")
def test_hot_kernels_do_not_spill(tmp_path):
    files = sorted({v[0] for v in KERNELS.values()})
    with ThreadPoolExecutor(max_workers=len(files)) as ex:
        texts = dict(zip(files, ex.map(lambda f: _assembly(f, str(tmp_path / (f[:-4] + ".s"))), files)))
    meta = {f: _metadata(t) for f, t in texts.items()}
    for key, (src, max_vgpr, max_lds) in KERNELS.items():
        hits = [(n, m) for n, m in meta[src].items() if key in n]
        assert len(hits) == 1, f"{key}: {len(hits)} kernels match in {src}"
        name, m = hits[0]
        assert m["vgpr_spill_count"] == 0 and m["private_segment_fixed_size"] == 0, f"{name} spills: {m}"
        assert m["vgpr_count"] + m["agpr_count"] <= max_vgpr, f"{name}: {m['vgpr_count']} + {m['agpr_count']} registers"
        assert m["group_segment_fixed_size"] <= max_lds, f"{name}: {m['group_segment_fixed_size']} bytes of LDS"


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not installed")
def test_boundary_search_reads_its_histogram_in_16_byte_pieces(tmp_path):
    """find_boundary opens every workgroup of the level kernels: eight bins per thread, two loads and no branch about them."""
    text = _assembly("k_select.hip", str(tmp_path / "k_select.s"))
    for level in (0, 1):
        body = re.search(r"^_Z16sel_level_kernelILi%dE.*?s_barrier" % level, text, re.M | re.S).group(0)
        assert len(re.findall(r"global_load_dwordx4", body)) == 2, body
        assert "global_load_dword " not in body and "s_cbranch" not in body, body


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not installed")
def test_gather_form_has_the_workgroups_that_run_at_once(tmp_path):
    """The gather form's even shares, S2_GATHER_BLOCKS of them, take one round of the chip's 256 compute units: as many per unit
    as the registers and the LDS of the 64-bit instances admit, no fewer (some units would hold more than others) and no more
    (a second round of few)."""
    meta = _metadata(_assembly("k_stage2.hip", str(tmp_path / "k_stage2.s")))
    defines = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-E", "-dD",
                              "--cuda-host-only", os.path.join(CSRC, "k_stage2.hip")], check=True, stdout=subprocess.PIPE,
                             stderr=subprocess.DEVNULL, text=True).stdout
    define = dict(re.findall(r"^#define (S2_GATHER_BLOCKS|S2_UNIT_BLOCKS)\s+(.*?)(?://.*)?$", defines, re.M))
    blocks = eval(define["S2_GATHER_BLOCKS"].strip(), {}, {k: int(v) for k, v in define.items() if v.strip().isdigit()})
    for key in ("s2_invert_kernelILi11EyLb0ELb0ELb0E", "s2_invert_kernelILi13EyLb0ELb0ELb0E", "s2_invert_kernelILi11EyLb0ELb1ELb0E",
                "s2_invert_kernelILi13EyLb0ELb1ELb0E"):
        m, = [m for n, m in meta.items() if key in n]
        vgprs = -(-(m["vgpr_count"] + m["agpr_count"]) // 8) * 8
        assert blocks == 256 * min(512 // vgprs, (160 << 10) // m["group_segment_fixed_size"]), (key, blocks, m)


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not installed")
def test_decompression_has_both_kinds_of_stores(tmp_path):
    """Vectors and indices are stored past the caches or through them, by a condition that is no part of the store: four rows a thread of each."""
    text = _assembly("k_stage4.hip", str(tmp_path / "k_stage4.s"))
    for nbits in (1, 2):
        body = re.search(r"^_Z22decompress_dump_kernelILi%dE.*?\.end_amdhsa_kernel" % nbits, text, re.M | re.S).group(0)
        for width in ("dwordx4", "dword"):
            stores = re.findall(r"global_store_%s (.*)" % width, body)
            assert len(stores) == 8 and sum(l.endswith(" nt") for l in stores) == 4, stores


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not installed")
def test_range_kernels_scalar_spills(tmp_path):
    """What only a single query (a key list in parts) or launches of fewer than 32 queries (duplicates among the probes) need is no state of the
    instances that never serve them: scalar registers spilled to vector ones, before they left those instances 106, 80, 142, 141."""
    meta = _metadata(_assembly("k_stage2.hip", str(tmp_path / "k_stage2.s")))
    for key, most in (("EjLb0ELb0ELb0E", 95), ("EjLb1ELb0ELb0E", 79), ("EyLb0ELb0ELb0E", 130), ("EyLb0ELb0ELb1E", 135), ("EyLb0ELb1E", 150)):
        spills = {n: m["sgpr_spill_count"] for n, m in meta.items() if "s2_invert_kernelILi" in n and key in n}
        assert spills and max(spills.values()) <= most, spills


# LDS arrays that are accessed in 16-byte pieces: (source file, where the array starts within the record it lies in)
LDS_PIECES = [
    ("k_scq.hip", ["offsetof(SurvivorRows, Qs)", "offsetof(SurvivorRows, row)", "offsetof(TableScratch<true>, x)",
                   "offsetof(ProbeScratch<true>, Qs)", "offsetof(ProbeScratch<true>, block)", "offsetof(ProbeScratch<true>, row)",
                   "offsetof(ProbeScratch<true>, idl)", "offsetof(ProbeScratch<false>, block)", "offsetof(ProbeScratch<false>, idl)"]),
    ("k_stage2.hip", ["offsetof(S2GatherScratch, list)", "offsetof(S2GatherScratch, part_max)"]),
    ("k_stage4.hip", ["offsetof(VpArea, code)", "offsetof(VpArea, end)", "sizeof(VpArea)", "offsetof(VpAreaOf<false>, code)",
                      "offsetof(VpAreaOf<false>, end)", "sizeof(VpAreaOf<false>)"]),
]


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not installed")
@pytest.mark.parametrize("src,places", LDS_PIECES, ids=[s for s, _ in LDS_PIECES])
def test_lds_arrays_accessed_in_16_byte_pieces_are_aligned(tmp_path, src, places):
    unit = tmp_path / "places.hip"
    unit.write_text(f'#include "{src}"\n#include <cstddef>\n' +
                    "".join(f'static_assert(({p}) % 16 == 0, "{p}");\n' for p in places))
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                        "--cuda-host-only", "-fsyntax-only", str(unit)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout


# What the rules that choose a kernel's form say on both sides of the lines that were measured: (source file, expression).
RULES = [
    # one query of 8.4, 8.8, 14 and 16, 20 million passages; two of 8.8; many
    ("k_stage2.hip", ["s2_steps(1, 4096) == 1", "s2_steps(1, 4297) == 2", "s2_steps(1, 6836) == 2", "s2_steps(1, 7813) == 1",
                      "s2_steps(1, 9766) == 1", "s2_steps(2, 8594) == 1", "s2_steps(512, 100352) == 2", "s2_steps(150, 644550) == 4",
                      # which of 32 (bit 0) to 63 survivors: a list in every range, in most of them, and where few need planes
                      "s2_tall_queries(1.0) == 0xFFE0001Fu", "s2_tall_queries(0.9999) == 0xFFE0001Fu", "s2_tall_queries(0.975) == 0xFFC0001Fu",
                      "s2_tall_queries(0.85) == 0xE00003FFu", "s2_tall_queries(0.71) == 0x0003FFF0u",
                      "s2_tall_queries(0.65) == 0", "s2_tall_queries(0.0) == 0",
                      # passages per range: smallest collections, those up to 400 ranges, large ones; many queries; large shares kept
                      "s2_range_log(1000, 1, 50) == 7", "s2_range_log(8192, 40, 100) == 7", "s2_range_log(8192, 41, 100) == 9", "s2_range_log(8193, 1, 256) == 9",
                      "s2_range_log(10000, 1, 500) == 8", "s2_range_log(10000, 16, 700) == 7", "s2_range_log(20000, 1, 1000) == 8", "s2_range_log(30000, 1, 2000) == 9", "s2_range_log(200000, 1, 256) == 9",
                      "s2_range_log(400000, 1, 1024) == 10", "s2_range_log(409601, 1, 1024) == 11", "s2_range_log(10000, 33, 256) == 9",
                      "s2_range_log(10000, 512, 256) == 11", "s2_range_log(40000, 1, 20000) == 7", "s2_range_log(400000, 1, 100000) == 9",
                      "s2_range_log(8800000, 1, 4096) == 11",
                      # first batches of whole and of shorter ranges; a share of ndocs that is more
                      "s2_first_batch(400000, 33, 256, 11) == 48", "s2_first_batch(400000, 32, 1024, 11) == 24", "s2_first_batch(8800000, 1, 4096, 11) == 48",
                      "s2_first_batch(400000, 1, 4096, 10) == 24", "s2_first_batch(30000, 64, 256, 9) == 24", "s2_first_batch(5000, 64, 256, 7) == 64", "s2_first_batch(400000, 1, 100000, 9) == 128",
                      "s2_first_batch(400000, 64, 40000, 11) == 204"]),
    # long lists in great number only
    ("k_stage4.hip", ["s4_packed(256, 512)", "s4_packed(1024, 36)", "!s4_packed(1024, 35)", "s4_packed(96, 384)", "!s4_packed(72, 512)",
                      "!s4_packed(64, 576)", "!s4_packed(64, 2048)", "!s4_packed(16, 2304)"]),
    # pruning by coarse scores (queries of a chunk, passages, candidates kept): the calls of test_gpu_vanilla_coarse.py
    ("plaid_api.hip", ["vanilla_screens(16, 70000, 17000)", "!vanilla_screens(16, 70000, 17501)", "vanilla_screens(16, 66000, 1)",
                       "vanilla_screens(6, 140000, 4096)", "!vanilla_screens(4, 140000, 4096)", "vanilla_screens(4, 200000, 3000)",
                       "vanilla_screens(16, 140001, 9000)", "vanilla_screens(8, 131072, 64)", "vanilla_screens(16, 52000, 13000)",
                       "vanilla_screens(16, 70000, 300)", "vanilla_screens(16, 70000, 2000)"]),
]


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not installed")
@pytest.mark.parametrize("src,claims", RULES, ids=[s for s, _ in RULES])
def test_rules_on_sizes(tmp_path, src, claims):
    unit = tmp_path / "rules.hip"
    unit.write_text(f'#include "{src}"\n' + "".join(f'static_assert({c}, "{c}");\n' for c in claims))
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                        "--cuda-host-only", "-fsyntax-only", str(unit)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not installed")
def test_half_exchanges_wait_for_their_operands(tmp_path):
    """v_permlane32_swap needs two wait states after a vector instruction that writes one of its operands.  The compiler sees to that,
    but for instructions in assembly statements, whose results the exchanges of k_stage4.hip take."""
    lines = [l.split(";")[0].strip() for l in _assembly("k_stage4.hip", str(tmp_path / "k_stage4.s")).splitlines()]
    lines = [l for l in lines if l and not l.startswith(".") and not l.endswith(":")]
    swaps = [i for i, l in enumerate(lines) if l.startswith("v_permlane32_swap")]
    assert swaps
    for i in swaps:
        operands = re.findall(r"v\d+", lines[i])
        states = 0
        for l in reversed(lines[max(0, i - 2):i]):
            if states >= 2:
                break
            op, _, rest = l.partition(" ")
            assert not (op.startswith("v_") and re.match(r"v\d+", rest.strip()) and re.match(r"v\d+", rest.strip()).group(0) in operands), lines[i - 4:i + 1]
            states += int(rest) + 1 if op == "s_nop" else 1
