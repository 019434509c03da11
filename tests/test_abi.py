"""CPU-side checks of the C-ABI library: it loads, exports every symbol include/isp.h declares,
and its argument checks that need no device work behave as documented."""
import ctypes
import os
import re

import pytest

import paper_2403_14853_amd as isp
from paper_2403_14853_amd import binding


def _header_symbols(repo_root):
    text = open(os.path.join(repo_root, "include", "isp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(isp_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol(repo_root):
    lib = isp.load_library()
    declared = _header_symbols(repo_root)
    assert declared, "no declarations found in include/isp.h"
    for name in declared:
        assert hasattr(lib, name), "libisp.so does not export %s" % name
    assert sorted(binding.EXPORTED_SYMBOLS) == declared
    assert lib.isp_version().decode().startswith("isp-gfx950")


def test_binding_names_follow_the_abi():
    for name in ("csr_build", "csr_transpose_cached", "spmm", "sddmm", "fusedmm", "fusedmm_backward"):
        assert callable(getattr(isp, name))


def test_argument_checks_without_device_work():
    lib = isp.load_library()
    need = ctypes.c_size_t()
    assert lib.isp_csr_build_workspace(10, 10, 20, None) == 1  # ISP_EINVAL
    assert b"NULL" in lib.isp_last_error()
    assert lib.isp_csr_build_workspace(-1, 10, 20, ctypes.byref(need)) == 1
    assert lib.isp_csr_build_workspace(10, 10, 2**31, ctypes.byref(need)) == 5  # ISP_EUNSUPPORTED
    assert lib.isp_csr_build_workspace(1000, 1000, 5000, ctypes.byref(need)) == 0 and need.value > 0
    small = need.value
    assert lib.isp_csr_build_workspace(100000, 100000, 5000000, ctypes.byref(need)) == 0 and need.value > small
    h = ctypes.c_void_p()
    assert lib.isp_csr_build(4, 4, 4, None, None, None, None, 0, 0, None, ctypes.byref(h)) == 1
    assert lib.isp_csr_build(4, 4, 4, None, None, None, None, 0, 0, None, None) == 1
    # NULL handles
    assert lib.isp_spmm(None, None, 4, 4, None, 4, None) == 1
    assert lib.isp_sddmm(None, None, 4, None, 4, 4, 0, None, None) == 1
    assert lib.isp_fusedmm(None, None, 4, 4, 0, None, 4, None) == 1
    assert lib.isp_fusedmm_backward(None, None, 4, None, 4, 4, 0, None, 4, None) == 1
    assert lib.isp_csr_transpose_workspace(None, ctypes.byref(need)) == 1
    assert lib.isp_csr_info(None, None) == 1
    lib.isp_csr_destroy(None)  # documented no-op


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_LIB_PATH", str(tmp_path / "libisp.so"))
    with pytest.raises(ImportError):
        binding.load_library()


def test_header_is_plain_c(repo_root, tmp_path):
    """include/isp.h is the boundary: it must compile as C99 on its own (no torch, no HIP, no C++)."""
    import subprocess
    src = tmp_path / "use_isp.c"
    src.write_text('#include "isp.h"\n'
                   "int main(void) {\n"
                   "  isp_csr_t* a = 0; size_t b = 0; isp_csr_info_t info;\n"
                   "  (void)info; (void)a;\n"
                   "  return isp_csr_build_workspace(1, 1, 1, &b) == ISP_OK ? 0 : 1;\n"
                   "}\n")
    subprocess.check_call(["gcc", "-std=c99", "-pedantic", "-Wall", "-Werror", "-fsyntax-only",
                           "-I", os.path.join(repo_root, "include"), str(src)])


def test_counter_records_parse_with_their_calibration():
    """profiles/counter_records.txt, which bench.py reads for roofline.traffic: the calibration lines are really
    lines of their own (FETCH_SIZE counts half the bytes on this part, so its factor is 2), every benchmark
    configuration has a record, and a record's bytes are at least the operands of its workload moved once."""
    import bench
    path = os.path.join(os.path.dirname(os.path.abspath(bench.__file__)), "profiles", "counter_records.txt")
    lines = [l.split("#")[0].split() for l in open(path)]
    factors = {f[0]: float(f[1]) for f in lines if len(f) == 2}
    assert factors == {"fetch_factor": 2.0, "write_factor": 1.0}
    shapes = {"c1-rmat169k-d128": (169343, 128), "c2-rmat233k-dense-d128": (232965, 128),
              "c3-rmat2.4m-d128": (2449029, 128), "c4-rmat1m-d64-fusedmm": (1 << 20, 64)}
    for workload, (n, d) in shapes.items():
        kernel = "k_fused_grouped<g_fwd>" if workload.startswith("c4") else "k_spmm_grouped"
        rec = bench.counter_record(workload, kernel)
        assert rec is not None and rec["commit"], workload
        assert rec["bytes"] == (2.0 * rec["fetch_kib"] + rec["write_kib"]) * 1024.0
        assert rec["bytes"] > 2 * 4.0 * n * d, (workload, rec["bytes"])  # X read and Y written at least once
        assert rec["write_kib"] * 1024.0 >= 4.0 * n * d * 0.95, workload   # Y is written whole


def test_counter_records_know_their_source(repo_root, tmp_path):
    """bench.py prints a record's traffic only for the source that was measured: comments do not count, code does, in the
    kernel's own unit, in the partition's and in the headers they include."""
    import shutil
    import bench
    src = os.path.join(repo_root, "paper_2403_14853_amd", "csrc")
    for kernel in ("k_spmm_grouped", "k_fused_grouped<g_fwd>"):
        ref = bench.source_digest(kernel)
        for name, counts in (("run_stream.h", True), ("csr_build.hip", True), ("partition_sizes.h", True), ("alias.hip", False)):
            copy = str(tmp_path / ("%s_%s" % (kernel[:8], name)))
            shutil.copytree(src, copy)
            path = os.path.join(copy, name)
            text = open(path).read()
            open(path, "w").write("// a remark\n" + text + "\n/* another\n   one */\n")
            assert bench.source_digest(kernel, copy) == ref
            open(path, "w").write(text + "\nstatic int planted;\n")
            assert (bench.source_digest(kernel, copy) != ref) == counts
    assert bench.source_digest("sddmm") is None
    rec = bench.counter_record("c3-rmat2.4m-d128", "k_spmm_grouped")
    assert rec["current"] in (True, False)


@pytest.mark.parametrize("n,nnz", [(2_449_029, 123_629_211), (232_965, 114_629_852), (1_000_000, 33_000_000), (70_000, 8_400_000),
                                   (100_000, 4_500_000), (60_000, 60_000_000), (4_000_000, 300_000_000), (60_000_000, 2_000_000_000)])
def test_room_for_copies_of_ragged_operands(n, nnz, monkeypatch):
    """What the copies add to the build workspace: nothing or little where the packed layout leaves partial rows idle, never
    more than 5 bytes per entry there and 128 MiB elsewhere."""
    for key in list(os.environ):
        if key.startswith("ISP_"):
            monkeypatch.delenv(key)
    with_copies = isp.csr_build_workspace(n, n, nnz)
    monkeypatch.setenv("ISP_STAGE_MIN", "0")
    extra = with_copies - isp.csr_build_workspace(n, n, nnz)
    packed = (8 << 20) <= nnz <= (256 << 20) and n >= 1 << 16
    assert 0 <= extra <= (5 * nnz if packed else (128 << 20))
    if packed and nnz >= 48 * n:
        assert extra == 0
