"""The build's check of the generated assembly of the tile kernels (paper_2512_15306_amd/build.py): the MFMAs are
written out as inline assembly, so nothing but MFMAs may touch accumulator registers between the first MFMA and the
wait states behind the K loop.  Here the check itself is tested, on hand-written assembly text."""
import os
import re
import shutil
import stat
import subprocess

import pytest

from paper_2512_15306_amd import build

NAME = "_ZN4llmq16gemm_tile_kernelILi0ELi0ELi4ELi4ELb0ENS_10GemmTuningELb0ELb0ELi0EEEvPKhS3_Pt"


def kernel(body: str, name: str = NAME) -> str:
    return "\t.text\n%s:                                ; @%s\n; %%bb.0:\n%s\n.Lfunc_end0:\n\t.size\t%s, .Lfunc_end0-%s\n" % (
        name, name, body, name, name)


GOOD = """\tv_mov_b32_e32 v5, 0
\tv_accvgpr_write_b32 a0, v5
\tv_accvgpr_write_b32 a1, v5
.LBB0_3:                                ; =>This Inner Loop Header: Depth=1
\tds_read_b128 v[10:13], v1
\ts_waitcnt lgkmcnt(0)
\tv_mfma_f32_16x16x128_f8f6f4 a[0:3], v[20:27], v[10:17], a[0:3]
\tbuffer_load_dwordx4 v2, s[8:11], s0 offen lds
\tv_mfma_f32_16x16x128_f8f6f4 a[4:7], v[20:27], v[10:17], a[4:7] blgp:1
\ts_cbranch_scc1 .LBB0_3
.LBB0_4:
\tv_accvgpr_write_b32 a8, v5
\tv_mfma_f32_16x16x128_f8f6f4 a[8:11], v[20:27], v[10:17], a[8:11]
\ts_nop 15
\ts_nop 15
\ts_waitcnt vmcnt(0)
\ts_barrier
\tv_accvgpr_read_b32 v30, a0
\tglobal_store_dwordx4 v[40:41], a[4:7], off
\ts_endpgm"""


def test_a_clean_kernel_passes():
    build.check_accumulator_reads("good.hip", kernel(GOOD))


@pytest.mark.parametrize("planted", [
    "\tv_accvgpr_read_b32 v30, a2",                                        # copy out of the accumulator file
    "\tscratch_store_dwordx4 off, a[4:7], off offset:16 ; 16-byte Folded Spill",
    "\tv_accvgpr_mov_b32 a9, a1",
    "\tscratch_load_dwordx4 a[0:3], off, off ; 16-byte Folded Reload",
    "\tv_accvgpr_write_b32 a3, 0",                                         # a constant the compiler re-creates
])
@pytest.mark.parametrize("where", ["in the loop", "behind the loop"])
def test_accumulator_access_inside_the_mfma_stretch_fails(planted, where):
    anchor = "\tbuffer_load_dwordx4 v2" if where == "in the loop" else "\ts_nop 15\n\ts_nop 15"
    bad = GOOD.replace(anchor, planted + "\n" + anchor, 1)
    assert bad != GOOD
    with pytest.raises(RuntimeError, match="accumulator registers touched"):
        build.check_accumulator_reads("bad.hip", kernel(bad))


# A tile with accumulators in ordinary registers as well; the path of a single K step zeroes them again behind the loop.
LARGE = GOOD.replace("a[8:11]", "v[48:51]").replace("\tv_accvgpr_write_b32 a8, v5\n", "").replace(".LBB0_4:\n", """\ts_branch .LBB0_4
.LBB0_2:
\tv_mov_b32_e32 v48, v5
\tv_mov_b64_e32 v[50:51], v[48:49]
\tv_accvgpr_write_b32 a0, v48
\ts_branch .LBB0_4
.LBB0_4:
""").replace("\tv_mov_b32_e32 v5, 0\n", "\tv_mov_b32_e32 v5, 0\n\tv_mov_b32_e32 v48, v5\n\ts_cbranch_scc0 .LBB0_2\n")


def test_accumulators_in_ordinary_registers_pass():
    assert "v[48:51], v[20:27]" in LARGE and ".LBB0_2:" in LARGE
    build.check_accumulator_reads("large.hip", kernel(LARGE))


@pytest.mark.parametrize("planted", ["\tv_mov_b32_e32 v60, v49", "\tv_mov_b32_e32 v49, v60", "\tscratch_store_dwordx4 off, v[48:51], off offset:16",
                                     "\tv_accvgpr_write_b32 a3, v50"])
@pytest.mark.parametrize("anchor", ["\tbuffer_load_dwordx4 v2", "\ts_cbranch_scc1 .LBB0_3", "\ts_nop 15\n\ts_nop 15"])
def test_ordinary_registers_that_hold_accumulators_are_checked_too(planted, anchor):
    with pytest.raises(RuntimeError, match="accumulator registers touched"):
        build.check_accumulator_reads("bad.hip", kernel(LARGE.replace(anchor, planted + "\n" + anchor, 1)))


def test_missing_wait_states_fail():
    with pytest.raises(RuntimeError, match="no wait states behind the last MFMA"):
        build.check_accumulator_reads("bad.hip", kernel(GOOD.replace("\ts_nop 15\n\ts_nop 15\n", "")))


def test_a_source_without_tile_kernels_fails():
    with pytest.raises(RuntimeError, match="no tile kernel found"):
        build.check_accumulator_reads("empty.hip", kernel(GOOD, name="_ZN4llmq19amax_partial_kernelEPKt"))


def test_kernels_without_mfma_are_skipped_but_others_still_count():
    adder = kernel("\tglobal_load_dwordx4 a[0:3], v[2:3], off\n\tv_accvgpr_read_b32 v1, a0\n\ts_endpgm", name=NAME.replace("Li0EEEv", "Li2EEEv"))
    build.check_accumulator_reads("mixed.hip", adder + kernel(GOOD))
    with pytest.raises(RuntimeError, match="no tile kernel found"):
        build.check_accumulator_reads("only_adder.hip", adder)


def failing_compiler(tmp_path, when):
    """A C++ compiler that fails if its command line holds `when`, and writes what it is asked for otherwise."""
    exe = tmp_path / "cxx"
    exe.write_text("#!/bin/sh\ncase \"$*\" in *%s*) echo no such luck; exit 1;; esac\nwhile [ \"$1\" != -o ]; do shift; done; echo module > \"$2\"\n" % when)
    exe.chmod(exe.stat().st_mode | stat.S_IXUSR)
    return str(exe)


@pytest.mark.parametrize("fails", ["binding.cpp", "-shared", "missing", None])
def test_the_library_does_not_need_the_module(fails, tmp_path, monkeypatch, capsys):
    """A module that does not compile or link, or has no compiler: the library is built and replaces the old one, and no module of
    another build stays beside it."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not found")
    lib, module = tmp_path / "libllmq.so", tmp_path / "_binding.so"
    lib.write_text("old")
    module.write_text("old")
    monkeypatch.setattr(build, "SOURCES", ["calibrate.hip"])
    monkeypatch.setattr(build, "CHECKED_SOURCES", set())
    monkeypatch.setattr(build, "LIB", str(lib))
    monkeypatch.setattr(build, "BINDING", str(module))
    monkeypatch.setenv("CXX", str(tmp_path / "nothing") if fails == "missing" else failing_compiler(tmp_path, fails or "never"))
    assert build.build() == str(lib)
    assert lib.read_bytes()[:4] == b"\x7fELF"
    if fails:
        assert not module.exists() and "FAILED: binding.cpp" in capsys.readouterr().err
    else:
        assert module.read_text() == "module\n"
    assert sorted(os.listdir(tmp_path)) == sorted(["libllmq.so"] + ([] if fails else ["_binding.so"]) + ([] if fails == "missing" else ["cxx"]))


def test_the_guarded_norm_of_wide_rows_fits_four_waves_to_a_simd(tmp_path):
    """Registers of rmsnorm_rows_kernel with guarded rows: 128 leave four waves to a SIMD.  (279, as it once had, were twice the time.)"""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not found")
    asm = tmp_path / "rmsnorm.s"
    subprocess.run([hipcc] + build.FLAGS + ["--cuda-device-only", "-S", os.path.join(build.CSRC, "rmsnorm.hip"), "-o", str(asm)], check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    counts = {m.group(1): int(m.group(2)) for m in re.finditer(r"\.amdhsa_kernel _ZN4llmq\d+rmsnorm_rows_kernelI(Lb[01]ELb1ELi\d+E)Lb.*?next_free_vgpr (\d+)", asm.read_text(), re.S)}
    assert len(counts) == 8 and max(counts.values()) <= 128, counts
