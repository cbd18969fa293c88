"""bench.py's roofline line and the committed counters: what a kernel's counters were taken of decides whether they count."""
import os
import shutil
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench
from paper_1910_11141_amd import workloads

CSRC = os.path.join(ROOT, "paper_1910_11141_amd", "csrc")


def roofline(monkeypatch, code):
    w = workloads.make(5, n_chains=16384, n_iters=2)
    monkeypatch.setattr(bench, "profile_json", lambda kind, kernel, name: {"bytes_per_grad_eval": 7000.0, "n_chains": 16384, "code": code}
                        if kind == "traffic" else None)
    return bench.roofline_of(w, workloads, {"variant": 3, "phase_ticks": [0, 0, 0]}, 10 ** 9, 1.0, True)


def test_traffic_counters_of_other_code_are_not_used(monkeypatch):
    now = bench.kernel_code_id("nuts_elem_kernel")
    r = roofline(monkeypatch, now)
    assert r["traffic"] == 7000.0 * 10 ** 9 and r["frac"] == 7000.0 / 8000.0       # of 8 TB/s
    for code in ("0" * 16, None):
        r = roofline(monkeypatch, code)
        assert r["traffic"] is None and r["frac"] is None and "traffic_note" in r  # (the basis fraction would be above 1)


def test_code_id_follows_the_code_of_all_headers_and_not_their_comments(tmp_path):
    csrc = str(tmp_path / "csrc")
    shutil.copytree(CSRC, csrc)
    ids = {k: bench.kernel_code_id(k, csrc) for k in bench.KERNEL_NAMES.values()}
    assert ids == {k: bench.kernel_code_id(k) for k in ids} and len(set(ids.values())) == len(ids)

    def append(name, text):
        with open(os.path.join(csrc, name), "a") as f:
            f.write(text)

    append("nuts_row.h", "\n// a remark  /* more */\n\n   /* and\n another */\n")
    assert ids == {k: bench.kernel_code_id(k, csrc) for k in ids}
    append("nuts_row.h", "namespace nuts { constexpr int kMore = 1; }\n")
    changed = {k for k in ids if bench.kernel_code_id(k, csrc) != ids[k]}
    assert changed == {"nuts_elem_kernel", "nuts_dense_kernel"}


def test_code_id_follows_the_flags_of_the_kernels_translation_units(monkeypatch):
    from paper_1910_11141_amd import build
    names = list(bench.KERNEL_NAMES.values()) + ["nuts_chip_kernel"]
    ids = {k: bench.kernel_code_id(k) for k in names}
    monkeypatch.setitem(build.EXTRA_FLAGS, "nuts_chip.hip", [])
    assert {k for k in names if bench.kernel_code_id(k) != ids[k]} == {"nuts_chip_kernel"}
    monkeypatch.setitem(build.EXTRA_FLAGS, "nuts_gauss.hip", [])
    assert {k for k in names if bench.kernel_code_id(k) != ids[k]} == {"nuts_chip_kernel", "nuts_quad_kernel", "nuts_elem_kernel"}
    monkeypatch.setattr(build, "FLAGS", build.FLAGS + ["-DMORE"])
    assert all(bench.kernel_code_id(k) != ids[k] for k in names)


def test_a_library_older_than_the_flags_is_stale(monkeypatch, tmp_path):
    from paper_1910_11141_amd import build
    lib = tmp_path / "lib.so"
    lib.write_bytes(b"")
    monkeypatch.setattr(build, "LIB_PATH", str(lib))
    monkeypatch.setattr(build, "sources", lambda: [])
    monkeypatch.setattr(build, "headers", lambda: [])
    flags = os.path.getmtime(build.__file__)
    for age, stale in ((-10, True), (10, False)):
        os.utime(lib, (flags + age, flags + age))
        assert build.is_stale() == stale
