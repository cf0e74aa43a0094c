"""bench.py's command-line contract on the host: it measures one GPU, so
--gpus N with N > 1 exits (status 2) with a message before touching a
GPU."""

import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"),
                        "--gpus", "2"], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 2
    assert "one GPU" in r.stderr
    assert r.stdout.strip() == ""


def test_counted_kernels_are_classed():
    """The counter summaries class every kernel of the diff pass by its name,
    demangled or not, and leave out the reference pass."""
    import bench
    for name, want in (
            ("void st::(anonymous namespace)::k_gather_conv<st::bf16_t, true, "
             "2, false, 3, 3>(st::ConvArgs)", "conv_gemm"),
            ("_ZN2st12_GLOBAL__N_113k_gather_convIDF16_Lb1ELi1ELb0ELi2ELi3EEEv"
             "NS_8ConvArgsE", "conv_gemm"),
            ("void st::k_conv_gemm_big<st::bf16_t>(st::ConvArgs)",
             "conv_gemm"),
            ("void st::k_conv_gemm<float, true, true, false, false, false>"
             "(st::ConvArgs)", None),
            ("void st::(anonymous namespace)::k_dense_conv<st::bf16_t, 0, 128,"
             " 128, 64, 32, 3, 0>(st::ConvArgs, int, int, int, int)", None),
            ("void st::k_compact<st::ListPred, 2>(unsigned long long const*)",
             "list_compact"),
            ("void st::k_chunk_scan_prep_rgb8<st::bf16_t>(st::ChunkScanArgs)",
             "chunk_scan_mask")):
        assert bench.kernel_class(name) == want, name


def test_kernel_hash_covers_every_kernel_source(tmp_path, monkeypatch):
    """A change to any source of the kernels changes the hash that counter
    summaries are matched by."""
    import shutil

    import bench
    csrc = os.path.join("paper_2410_20790_amd", "csrc")
    shutil.copytree(os.path.join(ROOT, csrc), tmp_path / csrc)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    seen = {bench.kernel_source_hash()}
    for f in sorted(os.listdir(tmp_path / csrc)):
        # the planner and the executor launch kernels, they hold none
        if f in ("st_plan.cpp", "st_exec.hip", "st_internal.h"):
            continue
        with open(tmp_path / csrc / f, "a") as out:
            out.write("//\n")
        h = bench.kernel_source_hash()
        assert h not in seen, f
        seen.add(h)
