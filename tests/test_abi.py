"""The C-ABI library: it loads, exports every symbol the header declares, and rejects bad arguments
on the host before touching a device.  No compute happens here."""
import ctypes as C
import os
import re
import subprocess
import sys

import numpy as np
import pytest

from paper_1910_11141_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions(header="nuts.h", prefix="nuts_"):
    text = open(os.path.join(ROOT, "include", header)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(" + prefix + r"[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    from paper_1910_11141_amd import pcvm
    lib = C.CDLL(B.LIB_PATH)
    for header, prefix, exports in (("nuts.h", "nuts_", B.EXPORTS), ("pcvm.h", "pcvm_", pcvm.EXPORTS)):
        names = declared_functions(header, prefix)
        assert set(names) == set(exports)
        for n in names:
            assert getattr(lib, n) is not None
    from paper_1910_11141_amd import ubench
    ulib = C.CDLL(ubench.LIB_PATH)
    names = declared_functions("nuts_ubench.h", "nuts_ubench_")
    assert names == ["nuts_ubench_circle_point", "nuts_ubench_exp_bounded", "nuts_ubench_fill", "nuts_ubench_last_error",
                     "nuts_ubench_log_unit", "nuts_ubench_logistic", "nuts_ubench_mfma_peak", "nuts_ubench_pair"]
    for n in names:
        assert getattr(ulib, n) is not None
    assert sorted(os.listdir(os.path.join(ROOT, "include"))) == ["nuts.h", "nuts_ubench.h", "pcvm.h"]


def test_struct_layouts_match_the_header():
    assert C.sizeof(B.nuts_target_desc) == 64
    assert C.sizeof(B.nuts_stats) == 72
    assert C.sizeof(B.nuts_sample_options) == 32


def test_create_target_rejects_bad_descriptors():
    lib = B.lib()
    out = C.c_void_p()
    assert lib.nuts_create_target(None, C.byref(out)) == B.NUTS_E_INVALID_ARG
    d = B.nuts_target_desc(0, 1, 2, None, None, None, None, 0, 1.0)
    assert lib.nuts_create_target(C.byref(d), None) == B.NUTS_E_INVALID_ARG
    for kw in [dict(kind=9), dict(kind=-1), dict(dtype=2), dict(dim=0), dict(kind=1), dict(kind=2), dict(kind=3)]:
        d = B.nuts_target_desc(0, 1, 2, None, None, None, None, 0, 1.0)
        for k, v in kw.items():
            setattr(d, k, v)
        assert lib.nuts_create_target(C.byref(d), C.byref(out)) == B.NUTS_E_INVALID_ARG, kw
        assert B.nuts_last_error()
    X = np.ones((3, 2)); y = np.array([0.0, 1.0, 2.0])
    with pytest.raises(B.NutsError) as e:
        B.Target(B.NUTS_TARGET_LOGISTIC_REGRESSION, 2, X=X, y=y)
    assert e.value.code == B.NUTS_E_INVALID_ARG and "y[2]" in str(e.value)
    with pytest.raises(B.NutsError):
        B.Target(B.NUTS_TARGET_LOGISTIC_REGRESSION, 2, X=X, y=np.zeros(3), prior_scale=0.0)
    with pytest.raises(B.NutsError):
        B.Target(B.NUTS_TARGET_GAUSS_DIAG, 2, scales=np.array([1.0, -1.0]))
    with pytest.raises(B.NutsError):
        B.Target(B.NUTS_TARGET_GAUSS_DENSE_PRECISION, 2, precision=np.array([[1.0, np.nan], [0.0, 1.0]]))


def test_sample_rejects_bad_arguments_before_touching_the_device():
    lib = B.lib()
    t = B.Target(B.NUTS_TARGET_STD_NORMAL, 2)     # needs no device
    good = dict(n_chains=4, n_iters=3, step_size=0.5, depth=6)
    for bad in [dict(n_chains=0), dict(n_iters=0), dict(step_size=0.0), dict(step_size=-1.0),
                dict(step_size=float("nan")), dict(step_size=float("inf")), dict(depth=0), dict(depth=21)]:
        a = dict(good); a.update(bad)
        rc = lib.nuts_sample(t.handle, a["n_chains"], a["n_iters"], a["step_size"], a["depth"], 1, None, None, None)
        assert rc == B.NUTS_E_INVALID_ARG, bad
    assert lib.nuts_sample(None, 4, 3, 0.5, 6, 1, None, None, None) == B.NUTS_E_INVALID_ARG
    opt = B.nuts_sample_options(None, 0, 7, 0)
    assert lib.nuts_sample_ex(t.handle, 4, 3, 0.5, 6, 1, C.byref(opt), None, None, None) == B.NUTS_E_INVALID_ARG
    opt = B.nuts_sample_options(None, -1, 0, 0)
    assert lib.nuts_sample_ex(t.handle, 4, 3, 0.5, 6, 1, C.byref(opt), None, None, None) == B.NUTS_E_INVALID_ARG
    opt = B.nuts_sample_options(None, 0, B.NUTS_VARIANT_TILE, 0)
    assert lib.nuts_sample_ex(t.handle, 4, 3, 0.5, 6, 1, C.byref(opt), None, None, None) == B.NUTS_E_UNSUPPORTED
    big = B.Target(B.NUTS_TARGET_STD_NORMAL, 5000)
    opt = B.nuts_sample_options(None, 0, B.NUTS_VARIANT_ELEM, 0)
    assert lib.nuts_sample_ex(big.handle, 4, 3, 0.5, 6, 1, C.byref(opt), None, None, None) == B.NUTS_E_UNSUPPORTED
    s = B.nuts_stats()
    assert lib.nuts_get_stats(t.handle, C.byref(s)) == B.NUTS_E_INVALID_ARG   # nothing has run
    assert lib.nuts_get_stats(None, C.byref(s)) == B.NUTS_E_INVALID_ARG
    assert lib.nuts_destroy_target(None) == B.NUTS_OK


def test_pcvm_layouts_and_program_validation_on_the_host():
    from paper_1910_11141_amd import pcvm, pcvm_programs as PP
    assert C.sizeof(pcvm.pcvm_program) == 40 and C.sizeof(pcvm.pcvm_stats) == 40
    assert PP.OP_DTYPE.itemsize == 32 and PP.BLOCK_DTYPE.itemsize == 32
    L = pcvm.lib()
    run = lambda p, batch=4, depth=8, steps=100: L.pcvm_run(C.byref(p) if p is not None else None, batch, None, depth,
                                                            steps, None, None, 0, None)
    assert run(None) == pcvm.PCVM_E_INVALID_ARG
    good = PP.fibonacci()
    # a well-formed table passes validation and then stops at the missing buffers, still on the host
    assert run(pcvm.describe(good)) == pcvm.PCVM_E_INVALID_ARG and "inputs" in pcvm.pcvm_last_error()
    def broken(field, index, value, table="ops"):
        P = PP.fibonacci()
        getattr(P, table)[field][index] = value
        return P
    cases = [broken("dst", 0, 99), broken("a", 1, -1), broken("fn", 0, 15), broken("kind", 2, 3),
             broken("term", 0, 4, "blocks"), broken("i", 0, 5, "blocks"), broken("j", 2, -1, "blocks"),
             broken("x", 0, 16, "blocks"), broken("first_op", 4, 9, "blocks"), broken("n_ops", 1, -1, "blocks")]
    for P in cases:
        assert run(pcvm.describe(P)) == pcvm.PCVM_E_INVALID_ARG
        assert "inputs" not in pcvm.pcvm_last_error()
    d = pcvm.describe(good)
    d.n_vars = 17
    assert run(d) == pcvm.PCVM_E_INVALID_ARG
    d = pcvm.describe(good)
    d.output_var = 5
    assert run(d) == pcvm.PCVM_E_INVALID_ARG


def test_no_cpu_fallback_without_a_gpu():
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    t = B.Target(B.NUTS_TARGET_STD_NORMAL, 2)
    with pytest.raises(B.NutsError) as e:
        B.nuts_sample(t, 4, 3, 0.5, 6, 1)
    assert e.value.code == B.NUTS_E_DEVICE
    with pytest.raises(B.NutsError) as e:
        B.Target(B.NUTS_TARGET_GAUSS_DIAG, 2, scales=np.ones(2))
    assert e.value.code == B.NUTS_E_DEVICE
    from paper_1910_11141_amd import pcvm, pcvm_programs as PP
    P = PP.fibonacci()
    fake = (C.c_int64 * 4)(1, 2, 3, 4)          # never dereferenced: the call stops at the missing device
    rc = pcvm.lib().pcvm_run(C.byref(pcvm.describe(P)), 4, fake, 8, 100, fake, None, 0, None)
    assert rc == pcvm.PCVM_E_DEVICE


def test_product_package_does_not_reference_the_oracle():
    pkg = os.path.join(ROOT, "paper_1910_11141_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".h", ".hip", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                assert "nuts_ref" not in text and "pcvm_ref" not in text, os.path.join(dirpath, f)
                assert not re.search(r"^\s*(from|import)\s+oracle", text, flags=re.M), os.path.join(dirpath, f)
                assert "oracle/" not in text, os.path.join(dirpath, f)


@pytest.mark.parametrize("sweep", ["throughput", "utilization", "pcvm"])
def test_measurement_modes_refuse_to_run_without_a_gpu(sweep):
    """The sweeps of bench.py are product code: no GPU, no numbers (and in particular no CPU stand-in)."""
    import subprocess
    import sys
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--sweep", sweep], cwd=ROOT, capture_output=True,
                       text=True, timeout=300)
    assert r.returncode != 0
    assert "GPU" in (r.stderr + r.stdout)


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], cwd=ROOT, capture_output=True, text=True,
                       timeout=300)
    assert r.returncode != 0 and "one GPU" in (r.stderr + r.stdout)


# ------------------------------------------------------------------ host logic: the tile variant's operand stream

def expected_tile_stream(X, y, lay):
    """The stream written out from the header's description of it, element by element."""
    n, d = X.shape
    ks1, mt, c = lay["ks1"], lay["mt"], lay["const_col"]
    pairs = (ks1 + 1) // 2 + 2 * mt
    Xs = X if c >= 0 else np.where(y[:, None] != 0, X, -X)

    def x(row, feat):
        return Xs[row, feat] if row < n and feat < d else 0.0

    out = np.zeros((lay["n_alloc_tiles"], pairs, 64, 2))
    for t in range(lay["n_alloc_tiles"]):
        for lane in range(64):
            for s in range(ks1):
                slot = 4 * s + lane // 16
                feat = slot if c < 0 else (d if slot >= d - 1 else (d - 1 if slot == c else slot))
                out[t, s // 2, lane, s % 2] = x(16 * t + lane % 16, feat)
            for u in range(mt):
                for s in range(4):
                    o = 2 * ((ks1 + 1) // 2) + 4 * u + s
                    out[t, o // 2, lane, o % 2] = x(16 * t + 4 * s + lane // 16, 16 * u + lane % 16)
    return out.reshape(-1)


def tile_case(n, d, seed, const=()):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, d))
    for col, value in const:
        X[:, col] = value
    y = (rng.random(n) < 0.5).astype(np.float64)
    return X, y


@pytest.mark.parametrize("n,d,const,want_col,want_ks1", [
    (37, 7, ((6, 1.0),), -1, 2),                 # d = 3 mod 4: a feature less saves no k-step, the column stays
    (50, 24, (), -1, 6),
    (50, 25, ((24, 1.0),), 24, 6),               # the data recipe: 24 features and a last column of ones
    (40, 9, ((3, -2.5),), 3, 2),                 # anywhere, any value
    (33, 9, ((2, 3.0), (6, -3.0)), 2, 2),        # the first of several
    (20, 9, ((3, 0.0),), -1, 3),                 # a column of zeros is an ordinary column
    (20, 9, ((3, np.inf),), -1, 3),              # and so is one that is not finite
    (16, 5, ((0, 0.5),), 0, 1),
    (1, 5, (), 0, 1),                            # one row: every column is constant, the first that is not zero goes
    (130, 29, ((28, 1.0),), 28, 7),
    (40, 17, ((16, 1.0),), 16, 4),               # 16 features left in the first GEMM, still two feature tiles
    (9, 1, ((0, 1.0),), -1, 1),                  # a single column stays where it is
])
def test_tile_operand_stream_on_the_host(n, d, const, want_col, want_ks1):
    """nuts_tile_pack runs nuts_create_target's packing without a device: which column (if any) leaves the first GEMM,
    the tile counts, and every element of the stream against the layout the header states."""
    X, y = tile_case(n, d, seed=n + d, const=const)
    lay, stream = B.nuts_tile_pack(X, y)
    tiles = -(-n // 16)
    assert lay["const_col"] == want_col and lay["ks1"] == want_ks1 and lay["mt"] == -(-d // 16)
    assert lay["const_val"] == (X[0, want_col] if want_col >= 0 else 0.0)
    assert lay["n_alloc_tiles"] == -(-tiles // 8) * 8
    assert lay["n_tiles"] == (tiles if want_col >= 0 else lay["n_alloc_tiles"])
    assert lay["n_pad"] == 16 * lay["n_tiles"] - n
    assert lay["operand_doubles"] == stream.size == lay["n_alloc_tiles"] * ((want_ks1 + 1) // 2 + 2 * lay["mt"]) * 128
    with np.errstate(invalid="ignore"):
        want = expected_tile_stream(X, y, lay)
    assert np.array_equal(stream, want, equal_nan=True)


def test_tile_pack_rejects_bad_arguments_on_the_host():
    X, y = tile_case(10, 33, seed=1)
    with pytest.raises(B.NutsError, match="range"):
        B.nuts_tile_pack(X, y)
    X, y = tile_case(10, 5, seed=1)
    lay = B.nuts_tile_layout()
    small = np.empty(8)
    rc = B.lib().nuts_tile_pack(X.ctypes.data_as(C.c_void_p), y.ctypes.data_as(C.c_void_p), C.c_int64(10), C.c_int64(5),
                                C.byref(lay), small.ctypes.data_as(C.c_void_p), C.c_int64(small.size))
    assert rc == B.NUTS_E_INVALID_ARG and "too small" in B.nuts_last_error()
    assert lay.operand_doubles > 8      # the layout is filled all the same
    rc = B.lib().nuts_tile_pack(None, y.ctypes.data_as(C.c_void_p), C.c_int64(10), C.c_int64(5), C.byref(lay), None, C.c_int64(0))
    assert rc == B.NUTS_E_INVALID_ARG


def test_out_of_host_memory_is_an_error_code_and_no_exception():
    """The packing of operands allocates on the host; in a process that may take little more memory that fails, and the
    call says so."""
    code = """
import resource, sys
import numpy as np
import paper_1910_11141_amd.binding as B
B.lib()
X, y = np.ones((400000, 25)), np.ones(400000)
X[::2] = 2.0
used = int(open('/proc/self/statm').read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (64 << 20), resource.RLIM_INFINITY))
lay = B.nuts_tile_layout()
import ctypes as C
rc = B.lib().nuts_tile_pack(X.ctypes.data_as(C.c_void_p), y.ctypes.data_as(C.c_void_p), C.c_int64(400000), C.c_int64(25), C.byref(lay), None, C.c_int64(0))
print(rc, B.nuts_last_error())
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-1000:]
    assert r.stdout.split()[:1] == [str(B.NUTS_E_ALLOC)] and "memory" in r.stdout
