"""Parity of the HIP path with the CPU oracle, through the C ABI, on a real MI355X.

Bar (from the benchmark definition): tree depths and leapfrog counts bit-exact in binary64 over the
first 50 iterations, states within 1e-10 relative (binary64) or 1e-4 (binary32, short runs).
"""
import json
import os

import numpy as np
import pytest

from oracle import nuts_ref as R
from paper_1910_11141_amd import workloads as W

pytestmark = pytest.mark.gpu

F64_TOL = 1e-10
F32_TOL = 1e-4


def N():
    import paper_1910_11141_amd.binding as B
    return B


def gpu_target(w, dtype=None):
    return N().Target(w.kind, w.dim, dtype or w.dtype, precision=w.precision, scales=w.scales, X=w.X, y=w.y,
                      prior_scale=w.prior_scale)


def ref_target(w, dtype=None):
    return R.Target(w.kind, w.dim, dtype or w.dtype, precision=w.precision, scales=w.scales, X=w.X, y=w.y,
                    prior_scale=w.prior_scale)


def gpu_run(w, variant=0, init=None, first_chain=0, n_chains=None, n_iters=None, tgt=None, leaf_steps=1, schedule=0,
            sampler=0):
    import torch
    B = N()
    tgt = tgt or gpu_target(w)
    nc, ni = n_chains or w.n_chains, n_iters or w.n_iters
    dev_init = None
    if init is not None:
        dev_init = torch.as_tensor(np.ascontiguousarray(init, dtype=w.dtype)).cuda()
    s, d, n = B.nuts_sample(tgt, nc, ni, w.step_size, w.max_tree_depth, w.seed, variant=variant,
                            init_states=dev_init, first_chain=first_chain, leaf_steps=leaf_steps,
                            schedule=schedule, sampler=sampler)
    torch.cuda.synchronize()
    return s.cpu().numpy(), d.cpu().numpy(), n.cpu().numpy(), B.nuts_get_stats(tgt)


def ref_run(w, chain_ids=None, init=None, n_chains=None, n_iters=None, leaf_steps=1, sampler=0):
    nc = len(chain_ids) if chain_ids is not None else (n_chains or w.n_chains)
    return R.sample(ref_target(w), nc, n_iters or w.n_iters, w.step_size, w.max_tree_depth, w.seed,
                    chain_ids=chain_ids, init_states=init, n_threads=8, want_margin=True, leaf_steps=leaf_steps,
                    sampler=sampler)


def state_error(gs, rs):
    """Largest error of any state component relative to that component's own scale: the oracle's largest
    magnitude of the same coordinate over the compared iterations and chains.  (A norm over all coordinates
    would let a coordinate of small scale be wrong by its whole size beside one of large scale.)"""
    if rs.size == 0:
        return 0.0
    scale = np.abs(rs).max(axis=(0, 1))
    scale = np.where(scale > 0, scale, 1.0)
    return float((np.abs(gs - rs) / scale).max())


def report(kind, **fields):
    """Measured agreement figures, one JSON line each, if NUTS_TEST_REPORT names a file (how the figures in the
    design notes were collected)."""
    path = os.environ.get("NUTS_TEST_REPORT")
    if path:
        with open(path, "a") as f:
            f.write(json.dumps(dict(kind=kind, test=os.environ.get("PYTEST_CURRENT_TEST", ""), **fields)) + "\n")


def assert_parity(gpu, ref, tol, cols=None, exact_ints=True, label=""):
    gs, gd, gn = gpu[:3]
    rs, rd, rn, margin = ref
    if cols is not None:
        gs, gd, gn = gs[:, cols], gd[:, cols], gn[:, cols]
    if exact_ints:
        bad = np.argwhere((gd != rd) | (gn != rn))
        assert bad.size == 0, f"{label}: integer outputs differ first at (iter, chain) {bad[0]}, " \
                              f"oracle decision margin there {margin[tuple(bad[0])]:.3e}"
    err = state_error(gs, rs)
    report("f64", label=label, err=err)
    assert err <= tol, f"{label}: states differ by {err:.3e} relative to their coordinate's scale (tolerance {tol})"
    return err


def check_invariants(w, d, n):
    assert (d >= 1).all() and (d <= w.max_tree_depth).all()
    assert (n >= 2 ** (d.astype(np.int64) - 1)).all() and (n <= 2 ** d.astype(np.int64) - 1).all()


# ------------------------------------------------------------------ the five configurations

def test_config1_std_normal_full():
    w = W.make(1)
    g = gpu_run(w)
    assert_parity(g, ref_run(w), F64_TOL, label=w.name)
    assert g[3]["leaf_slots_useful"] == g[2].sum()


def test_config2_dense_gaussian_full_chain_count_first_50_iterations():
    w = W.make(2, n_iters=50)
    g = gpu_run(w)
    check_invariants(w, g[1], g[2])
    ids = np.array([0, 1, 2, 3, 500, 777, 1022, 1023])
    assert_parity(g, ref_run(w, chain_ids=ids), F64_TOL, cols=ids, label=w.name)


def test_config3_logreg_full_chain_count_first_50_iterations_wave_kernel():
    w = W.make(3, n_iters=50)
    B = N()
    g = gpu_run(w, variant=B.NUTS_VARIANT_WAVE)
    check_invariants(w, g[1], g[2])
    assert np.isfinite(g[0]).all()
    ids = np.concatenate([np.arange(16), np.random.default_rng(0).choice(4096, 32, replace=False), [4095]])
    assert_parity(g, ref_run(w, chain_ids=ids), F64_TOL, cols=ids, label=w.name)
    st = g[3]
    assert st["leaf_slots_useful"] == g[2].sum() and st["extra_grad_evals"] == w.n_chains


def test_config4_large_logreg_f32_short_wave_kernel():
    w = W.make(4, n_chains=4, n_iters=4)
    g = gpu_run(w, variant=1)
    r = ref_run(w)
    # binary32 run: integer outputs are compared too, but a flipped decision is reported, not fatal
    f32_parity(g, r)


def test_config5_diag_gaussian_f32_short():
    w = W.make(5, n_chains=64, n_iters=20)
    g = gpu_run(w)
    r = ref_run(w)
    check_invariants(w, g[1], g[2])
    f32_parity(g, r)


# ------------------------------------------------------------------ ragged shapes and degenerate cases

@pytest.mark.parametrize("variant", [1, 3])
@pytest.mark.parametrize("dim", [1, 2, 3, 63, 64, 65, 130, 257, 512])
def test_std_normal_ragged_dimensions(dim, variant):
    w = W.Workload(f"std_d{dim}", W.STD_NORMAL, dim, np.dtype(np.float64), 9, 12, 0.35, 7, seed=5)
    g = gpu_run(w, variant=variant)
    assert g[3]["variant"] == variant
    assert_parity(g, ref_run(w), F64_TOL, label=w.name)


@pytest.mark.parametrize("dim", [1, 5, 64, 97])
def test_dense_gaussian_ragged_dimensions(dim):
    w = W.Workload(f"dense_d{dim}", W.GAUSS_DENSE, dim, np.dtype(np.float64), 7, 10, 0.2, 7, seed=6,
                   precision=W.random_spd_precision(dim, 3))
    assert_parity(gpu_run(w), ref_run(w), F64_TOL, label=w.name)


@pytest.mark.parametrize("dim,variant", [(1, 1), (1, 3), (66, 1), (66, 3), (129, 3), (500, 3), (1000, 1)])
def test_diag_gaussian_ragged_dimensions_f64(dim, variant):
    sig = 10.0 ** np.random.default_rng(dim).uniform(-1, 1, dim)
    w = W.Workload(f"diag_d{dim}", W.GAUSS_DIAG, dim, np.dtype(np.float64), 6, 8, 0.05, 8, seed=7, scales=sig)
    g = gpu_run(w, variant=variant)
    assert g[3]["variant"] == variant
    assert_parity(g, ref_run(w), F64_TOL, label=w.name)


@pytest.mark.parametrize("dim", [1, 5, 255, 256, 257, 1000, 1024])
def test_diag_gaussian_f32_register_kernel_is_bit_exact_on_short_runs(dim):
    """binary32 element-wise arithmetic is specified without fused multiply-add, reductions are binary64:
    over a few iterations the register kernel reproduces the oracle's integers exactly."""
    sig = (10.0 ** np.random.default_rng(dim).uniform(-1, 1, dim)).astype(np.float32)
    w = W.Workload(f"diag32_d{dim}", W.GAUSS_DIAG, dim, np.dtype(np.float32), 10, 6, 0.05, 8, seed=17, scales=sig)
    g = gpu_run(w, variant=3)
    r = ref_run(w)
    assert g[3]["variant"] == 3
    assert np.array_equal(g[1], r[1]) and np.array_equal(g[2], r[2])
    assert state_error(g[0], r[0]) <= F32_TOL


@pytest.mark.parametrize("n_data,dim", [(1, 1), (5, 2), (63, 3), (64, 16), (65, 17), (1000, 25), (257, 33), (300, 70)])
def test_logreg_ragged_shapes_wave_kernel(n_data, dim):
    w = W.small_logreg(n_data, dim, seed=100 + n_data)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 10, 12, 0.15 / np.sqrt(max(n_data, 1) / 10), 7
    B = N()
    assert_parity(gpu_run(w, variant=B.NUTS_VARIANT_WAVE), ref_run(w), F64_TOL, label=w.name)


def test_logreg_prior_scale_is_honoured():
    w = W.small_logreg(40, 4, seed=3)
    w.prior_scale = 2.5
    w.n_chains, w.n_iters = 6, 15
    B = N()
    assert_parity(gpu_run(w, variant=B.NUTS_VARIANT_WAVE), ref_run(w), F64_TOL, label="prior 2.5")


@pytest.mark.parametrize("variant", [1, 3])
def test_deep_trees_use_every_frame_level(variant):
    w = W.Workload("deep", W.STD_NORMAL, 2, np.dtype(np.float64), 5, 3, 0.004, 10, seed=8)
    g = gpu_run(w, variant=variant)
    r = ref_run(w)
    assert r[1].max() == 10 and r[2].max() == 1023
    assert_parity(g, r, F64_TOL, label="deep trees")


@pytest.mark.parametrize("variant", [1, 3])
def test_maximum_depth_limit_20_is_accepted(variant):
    w = W.Workload("cap20", W.STD_NORMAL, 3, np.dtype(np.float64), 4, 6, 0.3, 20, seed=9)
    assert_parity(gpu_run(w, variant=variant), ref_run(w), F64_TOL, label="max_tree_depth 20")


def test_depth_one_and_single_chain_single_iteration():
    w = W.Workload("d1", W.STD_NORMAL, 4, np.dtype(np.float64), 1, 1, 0.9, 1, seed=10)
    assert_parity(gpu_run(w), ref_run(w), F64_TOL, label="1x1, depth 1")
    w.n_chains, w.n_iters = 7, 25
    assert_parity(gpu_run(w), ref_run(w), F64_TOL, label="depth 1")


@pytest.mark.parametrize("variant", [1, 3])
def test_divergent_leaves_and_early_exits(variant):
    rng = np.random.default_rng(0)
    init = rng.standard_normal((12, 2)) * np.array([1.0, 40.0])
    w = W.Workload("div", W.STD_NORMAL, 2, np.dtype(np.float64), 12, 30, 1.75, 5, seed=5)
    g = gpu_run(w, init=init, variant=variant)
    r = ref_run(w, init=init)
    assert (r[2] != 2 ** r[1].astype(np.int64) - 1).sum() > 5      # partial trees do occur
    assert_parity(g, r, F64_TOL, label="divergent")


@pytest.mark.parametrize("variant", [1, 3])
def test_non_finite_energy_is_a_divergence_not_a_trap(variant):
    init = np.full((3, 2), 1e200)
    w = W.Workload("inf", W.STD_NORMAL, 2, np.dtype(np.float64), 3, 4, 0.5, 4, seed=2)
    g = gpu_run(w, init=init, variant=variant)
    r = ref_run(w, init=init)
    assert (g[1] == 1).all() and (g[2] == 1).all()
    assert np.array_equal(g[1], r[1]) and np.array_equal(g[2], r[2])
    assert np.array_equal(g[0], r[0])       # every proposal is rejected: the state never moves


def test_tile_kernel_logistic_function_is_accurate_to_rounding():
    import torch
    B = N()
    rng = np.random.default_rng(0)
    z = np.concatenate([rng.normal(scale=s, size=200000) for s in (0.1, 1.0, 5.0, 30.0)] +
                       [np.linspace(-70, 70, 100001), np.arange(0, 38 * 16 + 3) / 16.0,
                        np.nextafter(np.arange(1, 38 * 16 + 3) / 16.0, 0),
                        np.array([0.0, -0.0, 1e-300, 36.99, 37.0, 64.0, 745.0, 1e6, 1e300])])
    from paper_1910_11141_amd import ubench
    v, s = ubench.logistic(torch.as_tensor(z).cuda())
    v, s = v.cpu().numpy(), s.cpu().numpy()
    a = np.abs(z)
    want_v = 0.5 * a + np.log1p(np.exp(-a))
    assert (np.abs(v - want_v) <= 3e-16 * np.maximum(1.0, want_v)).all()
    assert np.abs(s - 0.5 * np.tanh(0.5 * a)).max() < 1e-15
    bad = np.array([np.nan, np.inf, -np.inf])
    v, s = ubench.logistic(torch.as_tensor(bad).cuda())
    assert not np.isfinite(v.cpu().numpy()).any()      # non-finite logits poison the log-density, never a trap
    # the logarithm of the product of sigmas (one per lane and round): products of up to 256 factors in [1/2, 1]
    x = np.concatenate([rng.uniform(0.5, 1.0, 200000), np.exp(-rng.uniform(0, 180, 200000)),
                        0.5 + (np.arange(0, 129) / 256.0), np.nextafter(0.5 + (np.arange(1, 129) / 256.0), 0),
                        2.0 ** -np.arange(0, 300), [1.0, np.nextafter(1.0, 0), 2.0 ** -256 * 1.999]])
    x = x[x <= 1.0]
    got = ubench.log_unit(torch.as_tensor(x).cuda()).cpu().numpy()
    want = np.log(x)
    assert (np.abs(got - want) <= 4.5e-16 * np.maximum(np.abs(want), 0.25)).all()   # 2 ulp; 1e-16 absolute next to x = 1
    assert np.isnan(ubench.log_unit(torch.as_tensor(np.array([np.nan])).cuda()).cpu().numpy()).all()
    # the sine and cosine of the Box-Muller draws: angles 2 pi u on a fine grid, at and next to every quarter turn
    quarter = np.arange(0, 5) * (np.pi / 2)
    phi = np.concatenate([2 * np.pi * rng.uniform(0, 1, 400000), 2 * np.pi * (np.arange(0, 4097) / 4096.0),
                          quarter, np.nextafter(quarter, 7.0)[:-1], np.nextafter(quarter, -1.0)[1:],
                          (np.arange(0, 8) + 0.5) * (np.pi / 4), [2.0 ** -53 * 2 * np.pi, 1e-300]])
    phi = phi[(phi >= 0) & (phi <= 2 * np.pi)]
    sn, cs = ubench.circle_point(torch.as_tensor(phi).cuda())
    # numpy's sin and cos are within an ulp of the true values; absolute next to a zero of the function, where
    # the angle's own rounding (2e-16 of a turn) is all there is
    assert np.abs(sn.cpu().numpy() - np.sin(phi)).max() <= 2.3e-16
    assert np.abs(cs.cpu().numpy() - np.cos(phi)).max() <= 2.3e-16
    # the exponential that makes a leaf's weight from its energy error: everyday errors, the whole range, the edges
    x = np.concatenate([rng.normal(0, 1, 300000), rng.uniform(-745, 700, 300000), np.arange(-1100, 701) * 1.0,
                        (np.arange(-1080, 1010) + 0.5) * np.log(2.0) / 1.0, [0.0, -0.0, 700.0, -745.2, -800.0, -1e300, -np.inf]])
    x = x[x <= 700.0]
    got = ubench.exp_bounded(torch.as_tensor(x).cuda()).cpu().numpy()
    want = np.exp(x)
    normal = want > 2.3e-308
    assert (np.abs(got[normal] - want[normal]) <= 3.4e-16 * want[normal]).all()     # 1.5 ulp
    assert (np.abs(got[~normal] - want[~normal]) <= 1e-323 + 3.4e-16 * want[~normal]).all()   # subnormal results and 0


# ------------------------------------------------------------------ tile kernel (8 chains in lock step, MFMA gradient)

def test_config3_logreg_full_chain_count_first_50_iterations_tile_kernel():
    w = W.make(3, n_iters=50)
    B = N()
    g = gpu_run(w, variant=B.NUTS_VARIANT_TILE)
    assert g[3]["variant"] == B.NUTS_VARIANT_TILE
    check_invariants(w, g[1], g[2])
    assert np.isfinite(g[0]).all()
    ids = np.concatenate([np.arange(16), np.random.default_rng(1).choice(4096, 48, replace=False), [4095]])
    assert_parity(g, ref_run(w, chain_ids=ids), F64_TOL, cols=ids, label=w.name)
    st = g[3]
    assert st["leaf_slots_useful"] == g[2].sum() and st["extra_grad_evals"] == w.n_chains
    assert st["leaf_slots_issued"] >= st["leaf_slots_useful"] + st["extra_grad_evals"]
    assert st["occupancy"] > 0.8


def test_auto_variant_picks_the_tile_kernel_for_config3():
    w = W.make(3, n_chains=64, n_iters=5)
    B = N()
    g = gpu_run(w)
    assert g[3]["variant"] == B.NUTS_VARIANT_TILE
    assert_parity(g, ref_run(w), F64_TOL, label="auto")


@pytest.mark.parametrize("n_data,dim", [(1, 1), (5, 2), (63, 3), (64, 16), (65, 17), (1000, 25), (129, 32), (2100, 31)])
def test_logreg_ragged_shapes_tile_kernel(n_data, dim):
    w = W.small_logreg(n_data, dim, seed=100 + n_data)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 21, 12, 0.15 / np.sqrt(max(n_data, 1) / 10), 7
    B = N()
    assert_parity(gpu_run(w, variant=B.NUTS_VARIANT_TILE), ref_run(w), F64_TOL, label=w.name)


def test_tile_kernel_many_rows_folds_the_product_of_sigmas():
    """More than 64 row tiles per wave (8192 rows): the running product of sigmas is folded into a logarithm between
    chunks of tiles; and 40 000 rows, where an unfolded product of up to 5000 factors per lane would underflow."""
    B = N()
    for n_data, n_chains in ((9000, 5), (40000, 3)):
        w = W.small_logreg(n_data, 4, seed=7 + n_data)
        w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = n_chains, 4, 0.15 / np.sqrt(n_data / 10), 5
        g = gpu_run(w, variant=B.NUTS_VARIANT_TILE)
        assert np.isfinite(g[0]).all()
        assert_parity(g, ref_run(w), F64_TOL, label=w.name)


@pytest.mark.parametrize("where,value", [("first", 1.0), ("middle", -2.5), ("none", 0.0), ("two", 3.0), ("zeros", 0.0)])
def test_tile_kernel_constant_column_anywhere_or_absent(where, value):
    """Columns that are the same in every row (the data recipe has one, the intercept): wherever they stand, whatever
    their value, and also when there is none, more than one, or one of zeros (which stays an ordinary column)."""
    w = W.small_logreg(77, 9, seed=31)
    X = w.X.copy()
    rng = np.random.default_rng(5)
    X[:, -1] = rng.standard_normal(77)             # no constant column left
    if where == "first":
        X[:, 0] = value
    elif where == "middle":
        X[:, 4] = value
    elif where == "two":
        X[:, 2] = value
        X[:, 6] = -value
    elif where == "zeros":
        X[:, 3] = 0.0
    w.X = X
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 19, 10, 0.05, 7
    B = N()
    assert_parity(gpu_run(w, variant=B.NUTS_VARIANT_TILE), ref_run(w), F64_TOL, label=f"constant column {where}")


@pytest.mark.parametrize("n_data,dim,col,value", [
    (1, 5, 0, 1.0), (7, 5, 4, 1.0), (16, 5, 2, -2.5), (128, 13, 12, 1.0), (131, 13, 0, 0.5), (300, 17, 16, 1.0),
    (129, 21, 7, 3.0), (2049, 29, 28, 1.0), (1000, 25, 0, 1.0), (40000, 5, 4, 1.0)])
def test_tile_kernel_constant_column_is_the_initial_value_of_the_first_gemm(n_data, dim, col, value):
    """With d = 1 mod 4 a constant column stays out of the first GEMM (one k-step less) and its share of every logit
    is the accumulators' initial value: every such d with both feature-tile counts, the column first, last and in
    between, row counts that fill the last tile, leave it ragged (its filler rows must start from zero, not from the
    column's share), give some waves no tile at all, and need the product of sigmas folded between chunks of tiles."""
    w = W.small_logreg(n_data, dim, seed=500 + n_data + dim)
    X = w.X.copy()
    X[:, -1] = np.random.default_rng(n_data).standard_normal(n_data)   # the recipe's own constant column goes
    X[:, col] = value
    w.X = X
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 19, 8, 0.15 / np.sqrt(max(n_data, 1) / 10), 6
    if n_data == 40000:
        w.n_chains, w.n_iters = 3, 4
    B = N()
    g = gpu_run(w, variant=B.NUTS_VARIANT_TILE)
    assert np.isfinite(g[0]).all()
    assert_parity(g, ref_run(w), F64_TOL, label=f"constant column {col} of {dim}, {n_data} rows")
    if n_data in (7, 131):
        assert_parity(gpu_run(w, variant=B.NUTS_VARIANT_TILE, sampler=1, leaf_steps=2), ref_run(w, sampler=1, leaf_steps=2),
                      F64_TOL, label="constant column, slice sampler")


def test_tile_kernel_deep_trees_and_depth_limit():
    w = W.small_logreg(30, 3, seed=4)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 18, 3, 0.002, 10
    B = N()
    g = gpu_run(w, variant=B.NUTS_VARIANT_TILE)
    r = ref_run(w)
    assert r[1].max() == 10 and r[2].max() == 1023
    assert_parity(g, r, F64_TOL, label="tile deep")
    w.max_tree_depth = 12
    w.n_iters = 1
    assert_parity(gpu_run(w, variant=B.NUTS_VARIANT_TILE), ref_run(w), F64_TOL, label="tile depth 12")


@pytest.mark.parametrize("dim", [4, 5])   # (5: the constant column is the first GEMM's initial value)
def test_tile_kernel_divergences_and_non_finite_states(dim):
    w = W.small_logreg(50, dim, seed=6)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 20, 20, 0.6, 6
    B = N()
    rng = np.random.default_rng(1)
    init = rng.standard_normal((20, dim)) * 5
    init[3] = 1e200
    init[7] = np.inf
    g = gpu_run(w, variant=B.NUTS_VARIANT_TILE, init=init)
    r = ref_run(w, init=init)
    assert (r[2] != 2 ** r[1].astype(np.int64) - 1).sum() > 5
    gs, rs = g[0].copy(), r[0].copy()
    assert np.array_equal(np.isfinite(gs), np.isfinite(rs))
    assert np.array_equal(g[1], r[1]) and np.array_equal(g[2], r[2])
    fin = np.isfinite(rs).all(axis=(0, 2))
    assert fin.sum() == 19 and not fin[7]
    assert state_error(gs[:, fin], rs[:, fin]) < F64_TOL


@pytest.mark.parametrize("scale, eps", [(60.0, 0.6), (300.0, 0.3)])
def test_tile_kernel_energy_far_below_the_start_moves_the_unit_of_the_weights(scale, eps):
    """The tile kernel keeps a trajectory's weights as numbers exp(H0 - H) in a unit that it moves when a leaf's energy
    falls more than 600 below it.  From starting points this far out (the prior term alone is -scale^2 d / 2) leapfrog
    steps of this size land hundreds to tens of thousands below the starting energy in the first trajectories (a plain
    numpy leapfrog of the same set-up shows it for 18 of 20 chains at scale 60 and for all at 300), and others diverge."""
    w = W.small_logreg(50, 4, seed=6)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 20, 10, eps, 6
    B = N()
    init = np.random.default_rng(1).standard_normal((20, 4)) * scale
    g = gpu_run(w, variant=B.NUTS_VARIANT_TILE, init=init)
    r = ref_run(w, init=init)
    assert_parity(g, r, F64_TOL, label=f"tile, start at {scale} sigma")
    for steps in (1, 3):
        assert_parity(gpu_run(w, variant=B.NUTS_VARIANT_TILE, init=init, leaf_steps=steps, sampler=1),
                      ref_run(w, init=init, leaf_steps=steps, sampler=1), F64_TOL, label="tile, far start, slice")


def test_tile_kernel_queues_chains_beyond_its_resident_slots_and_is_schedule_independent():
    w = W.small_logreg(40, 5, seed=8)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 9000, 3, 0.3, 5
    B = N()
    tgt = gpu_target(w)
    g = gpu_run(w, variant=B.NUTS_VARIANT_TILE, tgt=tgt)
    ids = np.array([0, 15, 16, 4097, 8191, 8192, 8999])
    assert_parity(g, ref_run(w, chain_ids=ids), F64_TOL, cols=ids, label="tile queue")
    small = gpu_run(w, variant=B.NUTS_VARIANT_TILE, tgt=tgt, n_chains=5)
    off = gpu_run(w, variant=B.NUTS_VARIANT_TILE, tgt=tgt, n_chains=33, first_chain=8000)
    again = gpu_run(w, variant=B.NUTS_VARIANT_TILE, tgt=tgt)
    for k in range(3):
        assert np.array_equal(g[k][:, :5], small[k])
        assert np.array_equal(g[k][:, 8000:8033], off[k])
        assert np.array_equal(g[k], again[k])


# ------------------------------------------------------------------ chip and grid kernels (binary32, rows spread over the chip)

def assert_chip(stats):
    """The run was the chip kernel's: the one kernel of its variant that has a phase clock."""
    assert stats["variant"] == N().NUTS_VARIANT_GRID and sum(stats["phase_ticks"]) > 0


def assert_grid(stats):
    """The run was the two-launch grid kernels'."""
    assert stats["variant"] == N().NUTS_VARIANT_GRID and sum(stats["phase_ticks"]) == 0


def f32_parity(g, r, min_agree=0.99, min_chains=0.95):
    """binary32: a decision that falls the other way in rounding changes a chain's whole future, so integer outputs
    are compared as a rate, and states on the chains whose decisions all agree (per coordinate, see state_error).
    Measured over every binary32 comparison of this file (131 of them, 1 to 1300 chains, up to 20 iterations): all
    integer outputs agree and no chain leaves the oracle's decisions; largest state error 2.0e-6.  The floors below
    leave room for one flipped decision in a hundred, not more."""
    same = (g[1] == r[1]) & (g[2] == r[2])
    ok = same.all(axis=0)
    err = state_error(g[0][:, ok], r[0][:, ok])
    report("f32", agree=float(same.mean()), chains_ok=float(ok.mean()), n_chains=int(ok.size), err=err)
    assert same.mean() >= min_agree, f"only {same.mean():.2%} of integer outputs agree"
    assert ok.sum() >= max(1, int(min_chains * ok.size)), f"only {ok.mean():.2%} of the chains never left the oracle's decisions"
    assert err <= F32_TOL, err


@pytest.mark.parametrize("n_data,dim,n_chains", [(5, 2, 3), (100, 7, 8), (1000, 33, 40), (3000, 100, 64),
                                                 (257, 128, 9), (4100, 65, 256), (31, 96, 5),
                                                 (600, 20, 129), (900, 40, 131), (2000, 100, 200),
                                                 (500, 72, 33), (700, 104, 17), (300, 97, 10)])
def test_logreg_f32_chip_kernel_ragged_shapes(n_data, dim, n_chains):
    w = W.small_logreg(n_data, dim, seed=200 + n_data, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = n_chains, 6, 0.15 / np.sqrt(max(n_data, 1) / 10), 6
    B = N()
    g = gpu_run(w, variant=B.NUTS_VARIANT_GRID)
    assert_chip(g[3])
    r = ref_run(w)
    check_invariants(w, g[1], g[2])
    f32_parity(g, r)
    assert g[3]["leaf_slots_useful"] == g[2].sum() and g[3]["extra_grad_evals"] == n_chains


def test_config4_large_logreg_f32_grid_kernels():
    w = W.make(4, n_chains=8, n_iters=10)
    g = gpu_run(w)
    assert_grid(g[3])                                  # chosen automatically for a chip-sized gradient
    f32_parity(g, ref_run(w))


def test_chip_kernel_is_schedule_independent_and_deterministic():
    w = W.small_logreg(2000, 20, seed=77, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 100, 5, 0.02, 6
    B = N()
    tgt = gpu_target(w)
    a = gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt)
    b = gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt)
    c = gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt, n_chains=37)
    o = gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt, n_chains=10, first_chain=50)
    assert_chip(a[3])
    for k in range(3):
        assert np.array_equal(a[k], b[k])
        assert np.array_equal(a[k][:, :37], c[k])
        assert np.array_equal(a[k][:, 50:60], o[k])


def test_chip_kernel_200_chains_equal_128_and_72():
    w = W.small_logreg(1500, 30, seed=78, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 200, 5, 0.03, 6
    B = N()
    tgt = gpu_target(w)
    a = gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt)
    b = gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt)
    lo = gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt, n_chains=128)
    hi = gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt, n_chains=72, first_chain=128)
    for k in range(3):
        assert np.array_equal(a[k], b[k])
        assert np.array_equal(a[k][:, :128], lo[k])
        assert np.array_equal(a[k][:, 128:], hi[k])
    st = a[3]
    assert_chip(st)
    assert st["leaf_slots_useful"] == a[2].sum() and st["leaf_slots_issued"] >= st["leaf_slots_useful"]


@pytest.mark.parametrize("n_chains", [700, 1300])
def test_chip_kernel_many_and_queued_chains(n_chains):
    # 700 chains: two or three a workgroup; 1300: more chains than the 1024 resident ones, the rest are queued
    w = W.small_logreg(800, 12, seed=79, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = n_chains, 4, 0.05, 5
    B = N()
    tgt = gpu_target(w)
    a = gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt)
    assert_chip(a[3])
    check_invariants(w, a[1], a[2])
    f32_parity(a, ref_run(w))
    assert a[3]["leaf_slots_useful"] == a[2].sum() and a[3]["extra_grad_evals"] == n_chains
    # which workgroup takes which chain depends on timing; the chains' results do not
    b = gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt)
    c = gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt, n_chains=300)
    for k in range(3):
        assert np.array_equal(a[k], b[k])
        assert np.array_equal(a[k][:, :300], c[k])
    both_schedules(w, B.NUTS_VARIANT_GRID)


# rows at the edges of a tile of 16, of the eight tiles of a step and of one, two and more slices; features at the edges of a
# feature tile and of a block of 16 bytes a lane; more chains than are resident
@pytest.mark.parametrize("n_data,dim,n_chains", [(1, 1, 1), (16, 16, 5), (17, 17, 33), (128, 4, 20), (129, 128, 6), (385, 112, 17), (1025, 3, 1030),
                                                 (2064, 48, 250), (40001, 2, 9)])
def test_chip_kernel_edges_match_the_oracle_on_both_schedules(n_data, dim, n_chains):
    B = N()
    w = W.small_logreg(n_data, dim, seed=300 + n_data + dim, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = n_chains, 4, 0.15 / np.sqrt(max(n_data, 1) / 10), 6
    tgt = gpu_target(w)
    free, sync = both_schedules(w, B.NUTS_VARIANT_GRID)
    assert_chip(free[3])
    f32_parity(free, ref_run(w))
    slice3 = gpu_run(w, tgt=tgt, variant=B.NUTS_VARIANT_GRID, sampler=SLICE, leaf_steps=3, n_iters=2)
    f32_parity(slice3, ref_run(w, sampler=SLICE, leaf_steps=3, n_iters=2))


def rows_summed_in_binary32(X, rows):
    """X' / 2 with one binary32 sum per `rows` consecutive rows, of fused multiply-adds in order, and binary64 sums of those."""
    n, d = X.shape
    x = np.concatenate([X, np.zeros((-n % rows, d), np.float32)]).reshape(-1, rows, d)
    acc = np.zeros(x.shape[::2], np.float32)
    for i in range(rows):
        acc = (acc.astype(np.float64) + 0.5 * x[:, i].astype(np.float64)).astype(np.float32)
    return acc.astype(np.float64).sum(axis=0)


@pytest.mark.parametrize("n_data,dim,rows", [(1500, 100, 32), (2040, 60, 32), (6000, 60, 64), (10000, 100, 64), (15000, 100, 64), (23000, 64, 96)])
def test_chip_kernel_gradients_are_as_exact_as_sums_of_few_rows(n_data, dim, rows):
    """The gradient at zero, where every residual is 1/2, out of the first leapfrog step of many chains that all start
    there: theta = v eps (r + v eps / 2 g), so every chain shows the same g, and roundings of its own that average out.
    The bar is one binary32 sum per 32 rows of fewer than 2048, else per 64 or a 256th of them, and binary64 beyond: what
    sums in the order of the grid kernels' row slices amount to.  (One sum per wave over up to 180 rows, and of four waves in
    binary32, is 1.1 to 1.4 times as far off.)"""
    rng = np.random.default_rng(n_data)
    X = np.concatenate([rng.standard_normal((n_data, dim - 1)), np.ones((n_data, 1))], axis=1).astype(np.float32)
    y = (rng.random(n_data) < 0.5).astype(np.float32)
    signed = np.where(y[:, None] != 0, X, -X)
    exact = 0.5 * signed.astype(np.longdouble).sum(axis=0)
    nc, eps = 1000, 2.0 ** round(np.log2(1.5 / np.sqrt(n_data)))
    w = W.Workload("at_zero", W.LOGREG, dim, np.dtype(np.float32), nc, 1, eps, 1, seed=43, X=X, y=y, prior_scale=1.0)
    s, _, n, st = gpu_run(w, variant=N().NUTS_VARIANT_GRID, init=np.zeros((nc, dim)))
    assert_chip(st)
    assert (n == 1).all()
    r0 = np.array([[z for i in range((dim + 1) // 2) for z in R.normal_pair(R.draw(w.seed, i, R.TAG_MOMENTUM, 0, 0, c))][:dim]
                   for c in range(nc)]).astype(np.float32).astype(np.float64)
    th = s[0].astype(np.float64)
    seen = np.stack([(th - v * eps * r0) * 2 / eps ** 2 for v in (1, -1)])
    off = np.abs(seen - exact.astype(np.float64)).max(axis=2)
    moved = np.abs(th).max(axis=1) > 0
    assert moved.sum() >= nc // 4
    pick = off.argmin(axis=0)
    g = seen[pick, np.arange(nc)][moved].mean(axis=0)
    err = float(np.sqrt(np.mean((g - exact.astype(np.float64)) ** 2)))
    bar = float(np.sqrt(np.mean((rows_summed_in_binary32(signed, rows).astype(np.float32) - exact.astype(np.float64)) ** 2)))
    report("at_zero", n=n_data, d=dim, err=err, bar=bar)
    assert err <= bar, f"error {err:.2e} against {bar:.2e}"


def chip_starts(tgt, refused=0, most_blocks=0):
    import ctypes as C
    B = N()
    B._check(B.lib().nuts_debug_chip_starts(tgt.handle, C.c_int(refused), C.c_int(most_blocks)))


def compute_units():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("n_data,dim,n_chains", [(300, 40, 9), (2064, 48, 250), (3000, 9, 1030), (10000, 100, 40), (23000, 64, 3), (700, 128, 5)])
def test_chip_kernel_with_fewer_workgroups_than_compute_units(n_data, dim, n_chains):
    """On part of the chip, where a workgroup has several slices of the rows and holds fewer chains, chains have the same bits."""
    w = W.small_logreg(n_data, dim, seed=500 + dim, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = n_chains, 2, 0.5 / np.sqrt(n_data), 4
    tgt = gpu_target(w)
    whole = gpu_run(w, tgt=tgt, variant=N().NUTS_VARIANT_GRID)
    assert_chip(whole[3])
    assert whole[3]["grid_blocks"] == min(compute_units(), 256)
    for most in (100, 31, 12, 7, 1):
        chip_starts(tgt, most_blocks=most)
        for kw in (dict(), dict(schedule=1)) if most == 12 else (dict(),):
            part = gpu_run(w, tgt=tgt, variant=N().NUTS_VARIANT_GRID, **kw)
            assert part[3]["grid_blocks"] == most and part[3]["leaf_slots_useful"] == part[2].sum()
            for k in range(3):
                assert np.array_equal(whole[k], part[k])


@pytest.mark.parametrize("refused", [1, 2, 3, 7])
def test_chip_kernel_starts_again_when_compute_units_are_taken(refused):
    """A start that not all workgroups reach is tried again, after three with half as many workgroups."""
    w = W.small_logreg(3000, 20, seed=83, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 300, 3, 0.02, 5
    tgt = gpu_target(w)
    want = gpu_run(w, tgt=tgt)
    for kw in (dict(), dict(schedule=1)):
        chip_starts(tgt, refused=refused)
        got = gpu_run(w, tgt=tgt, **kw)
        blocks = want[3]["grid_blocks"]
        for _ in range(refused // 3):
            blocks = (blocks + 1) // 2
        assert got[3]["grid_blocks"] == blocks
        for k in range(3):
            assert np.array_equal(want[k], got[k])
    again = gpu_run(w, tgt=tgt)
    assert again[3]["grid_blocks"] == want[3]["grid_blocks"]


def test_chip_kernel_waits_for_a_device_that_is_busy():
    """A run of another kernel that holds every compute unit, on another stream: the chip kernel's call takes longer, no more."""
    import torch
    B = N()
    busy = W.make(3, n_iters=4000)
    holder = gpu_target(busy)
    w = W.small_logreg(3000, 20, seed=83, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 300, 3, 0.02, 5
    tgt = gpu_target(w)
    want = gpu_run(w, tgt=tgt)
    first, second = torch.cuda.Stream(), torch.cuda.Stream()
    try:
        B.nuts_set_stream(first)
        with torch.cuda.stream(first):
            _, _, n_busy = B.nuts_sample(holder, busy.n_chains, busy.n_iters, busy.step_size, busy.max_tree_depth, busy.seed, want_states=False)
        B.nuts_set_stream(second)
        with torch.cuda.stream(second):
            got = gpu_run(w, tgt=tgt)
    finally:
        B.nuts_set_stream(None)
    torch.cuda.synchronize()
    for k in range(3):
        assert np.array_equal(want[k], got[k])
    assert B.nuts_get_stats(holder)["leaf_slots_useful"] == int(n_busy.sum(dtype=torch.int64))


def test_chip_kernel_on_a_stream_with_part_of_the_compute_units():
    import ctypes as C

    import torch
    B = N()
    w = W.small_logreg(10000, 100, seed=85, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 300, 3, 0.005, 5
    tgt = gpu_target(w)
    want = gpu_run(w, tgt=tgt)
    with open("/proc/self/maps") as f:
        hip = C.CDLL([line.split()[-1] for line in f if "libamdhip64" in line][0])
    cus = compute_units()
    words = (cus + 31) // 32
    mask = (C.c_uint32 * words)(*([0xffffffff] * (words // 2) + [0] * (words - words // 2)))
    raw = C.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(C.byref(raw), C.c_uint32(words), mask) == 0
    B.nuts_set_stream(raw.value)
    try:
        with torch.cuda.stream(torch.cuda.ExternalStream(raw.value)):
            got = gpu_run(w, tgt=tgt)
    finally:
        B.nuts_set_stream(None)
        torch.cuda.synchronize()
        hip.hipStreamDestroy(raw)
    assert got[3]["grid_blocks"] == words // 2 * 32
    for k in range(3):
        assert np.array_equal(want[k], got[k])


def test_chip_kernel_called_by_two_threads_at_once():
    """Runs of the chip kernel on one device take turns: two threads with a target and a stream each."""
    import threading

    import torch
    B = N()
    ws = []
    for n_data, dim in ((3000, 20), (6000, 60)):
        w = W.small_logreg(n_data, dim, seed=84, dtype=np.float32)
        w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 300, 4, 0.01, 5
        ws.append(w)
    want = [gpu_run(w) for w in ws]
    targets, got, failed = [gpu_target(w) for w in ws], [[], []], []

    def call(i):
        try:
            s = torch.cuda.Stream()
            B.nuts_set_stream(s)
            with torch.cuda.stream(s):
                for kw in (dict(), dict(schedule=1), dict()):
                    got[i].append(gpu_run(ws[i], tgt=targets[i], **kw))
        except Exception as e:  # noqa: BLE001
            failed.append(e)
        finally:
            B.nuts_set_stream(None)

    threads = [threading.Thread(target=call, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
    for i in range(2):
        for run in got[i]:
            for k in range(3):
                assert np.array_equal(want[i][k], run[k])


# large enough for the two-launch grid kernels: left-over features of one and two groups of 4, none, and the largest; from 65 505 rows on
# a slice's four runs of tiles, with one, two and more groups of columns in use
@pytest.mark.parametrize("n_data,dim,n_chains", [(46000, 33, 3), (15700, 97, 40), (12100, 17, 6), (24000, 71, 5), (12500, 128, 3), (12001, 32, 130),
                                                 (65504, 36, 3), (65505, 36, 35), (65600, 128, 3), (70001, 24, 66), (66000, 72, 97)])
def test_grid_kernels_on_many_rows_match_the_oracle(n_data, dim, n_chains):
    w = W.small_logreg(n_data, dim, seed=400 + dim, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = n_chains, 2, 0.5 / np.sqrt(n_data), 4
    g = gpu_run(w)
    assert_grid(g[3])
    assert g[3]["leaf_slots_useful"] == g[2].sum()
    f32_parity(g, ref_run(w))
    few = gpu_run(w, n_chains=2)
    for k in range(3):
        assert np.array_equal(g[k][:, :2], few[k])


# just above the chip kernel's line: one set of columns, one set on each of two streams (129 chains), two sets a stream with columns
# handed out, and more chains than are resident; the last target's slices are four runs of tiles
@pytest.mark.parametrize("n_data,dim,n_chains", [(12001, 17, 40), (12001, 17, 129), (12001, 17, 260), (12001, 17, 1100), (24000, 71, 9), (24000, 71, 300),
                                                 (65505, 36, 260)])
def test_grid_kernels_slice_sampler_several_steps_a_leaf_and_both_schedules(n_data, dim, n_chains):
    B = N()
    w = W.small_logreg(n_data, dim, seed=420 + dim, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = n_chains, 3, 0.3 / np.sqrt(n_data), 3
    pick = np.unique(np.array([0, 1, n_chains // 2, n_chains - 1]))
    for kw in (dict(), dict(sampler=SLICE, leaf_steps=3)):
        free, sync = both_schedules(w, B.NUTS_VARIANT_GRID, **kw)
        assert_grid(free[3])
        assert_grid(sync[3])
        f32_parity([x[:, pick] for x in free[:3]], ref_run(w, chain_ids=pick, **kw))
        few = gpu_run(w, n_chains=6, first_chain=n_chains - 6, **kw)
        for k in range(3):
            assert np.array_equal(free[k][:, n_chains - 6:], few[k])


# ------------------------------------------------------------------ independence of the schedule

def test_chain_results_do_not_depend_on_batch_size_or_slot():
    """Section 2 of the paper: a batch member's execution is what it would be alone."""
    w = W.make(3, n_chains=300, n_iters=6)
    tgt = gpu_target(w)
    B = N()
    big = gpu_run(w, variant=B.NUTS_VARIANT_WAVE, tgt=tgt)
    small = gpu_run(w, variant=B.NUTS_VARIANT_WAVE, tgt=tgt, n_chains=7)
    off = gpu_run(w, variant=B.NUTS_VARIANT_WAVE, tgt=tgt, n_chains=20, first_chain=100)
    again = gpu_run(w, variant=B.NUTS_VARIANT_WAVE, tgt=tgt)
    for k in range(3):
        assert np.array_equal(big[k][:, :7], small[k])
        assert np.array_equal(big[k][:, 100:120], off[k])
        assert np.array_equal(big[k], again[k])


def test_more_chains_than_resident_slots_are_queued():
    w = W.Workload("queue", W.STD_NORMAL, 8, np.dtype(np.float64), 20000, 2, 0.4, 5, seed=11)
    g = gpu_run(w)
    ids = np.array([0, 1, 4999, 12345, 19999])
    assert_parity(g, ref_run(w, chain_ids=ids), F64_TOL, cols=ids, label="queued chains")
    assert g[3]["leaf_slots_useful"] == g[2].sum() and g[3]["extra_grad_evals"] == 20000


def test_null_outputs_are_allowed():
    import torch
    B = N()
    w = W.make(1)
    tgt = gpu_target(w)
    d = torch.empty((w.n_iters, w.n_chains), dtype=torch.int32, device="cuda")
    B._check(B.lib().nuts_sample(tgt.handle, w.n_chains, w.n_iters, w.step_size, w.max_tree_depth, w.seed,
                                 None, d.data_ptr(), None))
    torch.cuda.synchronize()
    assert np.array_equal(d.cpu().numpy(), ref_run(w)[1])


def test_runs_on_a_caller_stream():
    import torch
    B = N()
    w = W.make(1)
    s = torch.cuda.Stream()
    B.nuts_set_stream(s)
    try:
        with torch.cuda.stream(s):
            g = gpu_run(w)
    finally:
        B.nuts_set_stream(None)
    assert_parity(g, ref_run(w), F64_TOL, label="stream")


@pytest.mark.parametrize("n_data,dim,which", [(700, 10, assert_chip), (12001, 17, assert_grid)])
def test_chip_and_grid_kernels_on_a_caller_stream_back_to_back_calls(n_data, dim, which):
    # calls of different sizes in a row on a caller's stream must equal the same calls on the default stream: the workspace
    # grows between them, and the grid kernels fork to streams of their own and join them to the caller's
    import torch
    B = N()
    w = W.small_logreg(n_data, dim, seed=81, dtype=np.float32)
    w.n_iters, w.step_size, w.max_tree_depth = 4, 1.3 / np.sqrt(n_data), 5
    tgt = gpu_target(w)
    ref = [gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=gpu_target(w), n_chains=c) for c in (40, 600, 130)]
    s = torch.cuda.Stream()
    B.nuts_set_stream(s)
    try:
        with torch.cuda.stream(s):
            got = [gpu_run(w, variant=B.NUTS_VARIANT_GRID, tgt=tgt, n_chains=c) for c in (40, 600, 130)]
    finally:
        B.nuts_set_stream(None)
    for a, b in zip(ref, got):
        which(a[3])
        which(b[3])
        for k in range(3):
            assert np.array_equal(a[k], b[k])


# ------------------------------------------------------------------ several leapfrog steps per leaf (Section 4.1 uses 4)

def check_leaf_invariants(w, d, n, k):
    leaves = n // k
    assert (n % k == 0).all()
    assert (leaves >= 2 ** (d.astype(np.int64) - 1)).all() and (leaves <= 2 ** d.astype(np.int64) - 1).all()


@pytest.mark.parametrize("k", [2, 4, 7])
@pytest.mark.parametrize("variant", [1, 3])
def test_leaf_steps_std_normal_and_diag(variant, k):
    w = W.Workload(f"std_k{k}", W.STD_NORMAL, 67, np.dtype(np.float64), 9, 12, 0.35 / k, 7, seed=50 + k)
    g = gpu_run(w, variant=variant, leaf_steps=k)
    assert g[3]["variant"] == variant and g[3]["leaf_slots_useful"] == g[2].sum()
    check_leaf_invariants(w, g[1], g[2], k)
    assert_parity(g, ref_run(w, leaf_steps=k), F64_TOL, label=w.name)
    sig = 10.0 ** np.random.default_rng(k).uniform(-1, 1, 130)
    w = W.Workload(f"diag_k{k}", W.GAUSS_DIAG, 130, np.dtype(np.float64), 6, 8, 0.05 / k, 8, seed=7, scales=sig)
    assert_parity(gpu_run(w, variant=variant, leaf_steps=k), ref_run(w, leaf_steps=k), F64_TOL, label=w.name)


def test_leaf_steps_dense_gaussian_config2_paper_setting():
    """Configuration 2 at the paper's own leaf size: 4 leapfrog steps per leaf."""
    w = W.make(2, n_chains=24, n_iters=20)
    w.step_size = w.step_size / 2
    g = gpu_run(w, leaf_steps=4)
    check_leaf_invariants(w, g[1], g[2], 4)
    assert_parity(g, ref_run(w, leaf_steps=4), F64_TOL, label="config 2, 4 steps per leaf")


@pytest.mark.parametrize("k", [2, 4])
@pytest.mark.parametrize("n_data,dim", [(65, 17), (1000, 25), (129, 32)])
def test_leaf_steps_logreg_tile_and_wave_kernels(n_data, dim, k):
    w = W.small_logreg(n_data, dim, seed=100 + n_data)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 21, 12, 0.3 / k / np.sqrt(max(n_data, 1) / 10), 7
    B = N()
    r = ref_run(w, leaf_steps=k)
    assert len(np.unique(r[1])) >= 2
    for variant in (B.NUTS_VARIANT_TILE, B.NUTS_VARIANT_WAVE):
        g = gpu_run(w, variant=variant, leaf_steps=k)
        assert g[3]["variant"] == variant and g[3]["leaf_slots_useful"] == g[2].sum()
        check_leaf_invariants(w, g[1], g[2], k)
        assert_parity(g, r, F64_TOL, label=f"{w.name} variant {variant} k={k}")


def test_leaf_steps_config3_tile_kernel_at_full_chain_count():
    w = W.make(3, n_iters=20)
    w.step_size = w.step_size / 2
    B = N()
    g = gpu_run(w, variant=B.NUTS_VARIANT_TILE, leaf_steps=4)
    check_leaf_invariants(w, g[1], g[2], 4)
    ids = np.concatenate([np.arange(8), np.random.default_rng(2).choice(4096, 24, replace=False), [4095]])
    assert_parity(g, ref_run(w, chain_ids=ids, leaf_steps=4), F64_TOL, cols=ids, label="config 3, 4 steps per leaf")


def test_leaf_steps_with_divergences_tile_kernel():
    w = W.small_logreg(50, 4, seed=6)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 20, 20, 0.45, 6
    B = N()
    init = np.random.default_rng(1).standard_normal((20, 4)) * 5
    g = gpu_run(w, variant=B.NUTS_VARIANT_TILE, init=init, leaf_steps=2)
    r = ref_run(w, init=init, leaf_steps=2)
    assert (r[2] // 2 != 2 ** r[1].astype(np.int64) - 1).sum() > 5
    assert_parity(g, r, F64_TOL, label="tile divergent k=2")


@pytest.mark.parametrize("n_data,dim,n_chains,k", [(100, 7, 8, 2), (1000, 33, 40, 4), (257, 128, 9, 3)])
def test_leaf_steps_logreg_f32_chip_kernel(n_data, dim, n_chains, k):
    w = W.small_logreg(n_data, dim, seed=200 + n_data, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = n_chains, 6, 0.3 / k / np.sqrt(max(n_data, 1) / 10), 6
    B = N()
    g = gpu_run(w, variant=B.NUTS_VARIANT_GRID, leaf_steps=k)
    assert_chip(g[3])
    assert g[3]["leaf_slots_useful"] == g[2].sum()
    check_leaf_invariants(w, g[1], g[2], k)
    f32_parity(g, ref_run(w, leaf_steps=k))


def test_leaf_steps_argument_is_validated():
    B = N()
    t = B.Target(W.STD_NORMAL, 3, np.float64)
    for bad in (-1, 65):
        with pytest.raises(B.NutsError):
            B.nuts_sample(t, 2, 2, 0.1, 3, 1, leaf_steps=bad)


# ------------------------------------------------------------------ trajectory-synchronised schedule (Section 4.2)

def both_schedules(w, variant, **kw):
    B = N()
    tgt = gpu_target(w)
    free = gpu_run(w, variant=variant, tgt=tgt, schedule=B.NUTS_SCHEDULE_FREE, **kw)
    sync = gpu_run(w, variant=variant, tgt=tgt, schedule=B.NUTS_SCHEDULE_TRAJECTORY, **kw)
    assert free[3]["variant"] == sync[3]["variant"] == variant
    for a, b in zip(free[:3], sync[:3]):
        assert np.array_equal(a, b)             # the schedule must not show in the outputs
    n_chains, n_iters = free[1].shape[1], free[1].shape[0]
    assert free[3]["extra_grad_evals"] == n_chains
    assert sync[3]["extra_grad_evals"] == n_chains * n_iters
    assert sync[3]["leaf_slots_useful"] == free[3]["leaf_slots_useful"] == free[2].sum()
    return free, sync


@pytest.mark.parametrize("variant", [1, 3])
def test_schedules_agree_std_normal_and_diag(variant):
    w = W.Workload("std_sync", W.STD_NORMAL, 67, np.dtype(np.float64), 9, 12, 0.35, 7, seed=61)
    free, sync = both_schedules(w, variant)
    assert_parity(sync, ref_run(w), F64_TOL, label="std normal, trajectory schedule")
    sig = (10.0 ** np.random.default_rng(3).uniform(-1, 1, 300)).astype(np.float32)
    w = W.Workload("diag32_sync", W.GAUSS_DIAG, 300, np.dtype(np.float32), 10, 6, 0.05, 8, seed=17, scales=sig)
    both_schedules(w, variant)


def test_schedules_agree_dense_gaussian_and_occupancy_drops():
    """Figure 7's point: waiting at trajectory boundaries wastes gradient slots, batching across them does not."""
    w = W.make(2, n_chains=64, n_iters=10)
    free, sync = both_schedules(w, 1)
    assert_parity(sync, ref_run(w), F64_TOL, label="config 2, trajectory schedule")
    nl = free[2].astype(np.int64)
    # one chain per slot: the launch lasts as long as its busiest chain
    want_sync = nl.sum() / (64 * (nl.max(axis=1) + 1).sum())
    want_free = nl.sum() / (64 * (nl.sum(axis=0) + 1).max())
    assert abs(sync[3]["occupancy"] - want_sync) < 1e-12
    assert abs(free[3]["occupancy"] - want_free) < 1e-12
    assert sync[3]["occupancy"] < free[3]["occupancy"]


@pytest.mark.parametrize("n_data,dim", [(65, 17), (1000, 25)])
def test_schedules_agree_logreg_tile_and_wave_kernels(n_data, dim):
    w = W.small_logreg(n_data, dim, seed=100 + n_data)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 37, 9, 0.15 / np.sqrt(max(n_data, 1) / 10), 7
    B = N()
    r = ref_run(w)
    for variant in (B.NUTS_VARIANT_TILE, B.NUTS_VARIANT_WAVE):
        free, sync = both_schedules(w, variant)
        assert_parity(sync, r, F64_TOL, label=f"logreg variant {variant}, trajectory schedule")
    assert sync[3]["occupancy"] <= 1.0


def test_schedules_agree_logreg_f32_chip_kernel():
    w = W.small_logreg(1000, 33, seed=1200, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 12, 5, 0.015, 6
    B = N()
    free, sync = both_schedules(w, B.NUTS_VARIANT_GRID)
    assert_chip(free[3])
    assert_chip(sync[3])


def test_trajectory_schedule_with_leaf_steps_init_states_offsets_and_no_state_output():
    import torch
    B = N()
    w = W.small_logreg(200, 6, seed=77)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 19, 7, 0.05, 6
    init = np.random.default_rng(4).standard_normal((19, 6))
    free, sync = both_schedules(w, B.NUTS_VARIANT_TILE, init=init, first_chain=1000, leaf_steps=3)
    tgt = gpu_target(w)
    s, d, n = B.nuts_sample(tgt, 19, 7, w.step_size, w.max_tree_depth, w.seed, variant=B.NUTS_VARIANT_TILE,
                            init_states=torch.as_tensor(init).cuda(), first_chain=1000, leaf_steps=3,
                            schedule=B.NUTS_SCHEDULE_TRAJECTORY, want_states=False)
    torch.cuda.synchronize()
    assert s is None
    assert np.array_equal(d.cpu().numpy(), free[1]) and np.array_equal(n.cpu().numpy(), free[2])
    with pytest.raises(B.NutsError):
        B.nuts_sample(tgt, 2, 2, 0.1, 3, 1, schedule=2)


# ------------------------------------------------------------------ slice-sampling form (the published algorithm)

SLICE = 1


@pytest.mark.parametrize("variant", [1, 3])
def test_slice_sampler_std_normal_diag_and_deep_trees(variant):
    w = W.Workload("std_slice", W.STD_NORMAL, 67, np.dtype(np.float64), 9, 12, 0.35, 7, seed=71)
    g = gpu_run(w, variant=variant, sampler=SLICE)
    r = ref_run(w, sampler=SLICE)
    assert g[3]["variant"] == variant
    assert_parity(g, r, F64_TOL, label="std normal, slice")
    assert not np.array_equal(r[0], ref_run(w)[0])
    sig = 10.0 ** np.random.default_rng(9).uniform(-1, 1, 130)
    w = W.Workload("diag_slice", W.GAUSS_DIAG, 130, np.dtype(np.float64), 6, 8, 0.05, 8, seed=7, scales=sig)
    assert_parity(gpu_run(w, variant=variant, sampler=SLICE), ref_run(w, sampler=SLICE), F64_TOL, label="diag, slice")
    w = W.Workload("deep_slice", W.STD_NORMAL, 2, np.dtype(np.float64), 5, 3, 0.004, 10, seed=8)
    r = ref_run(w, sampler=SLICE)
    assert r[1].max() == 10 and r[2].max() == 1023
    assert_parity(gpu_run(w, variant=variant, sampler=SLICE), r, F64_TOL, label="deep trees, slice")


@pytest.mark.parametrize("variant", [1, 3])
def test_slice_sampler_divergences_and_non_finite_energy(variant):
    init = np.random.default_rng(0).standard_normal((12, 2)) * np.array([1.0, 40.0])
    w = W.Workload("div_slice", W.STD_NORMAL, 2, np.dtype(np.float64), 12, 30, 1.75, 5, seed=5)
    r = ref_run(w, init=init, sampler=SLICE)
    assert (r[2] != 2 ** r[1].astype(np.int64) - 1).sum() > 5
    assert_parity(gpu_run(w, init=init, variant=variant, sampler=SLICE), r, F64_TOL, label="divergent, slice")
    init = np.full((3, 2), 1e200)
    w = W.Workload("inf_slice", W.STD_NORMAL, 2, np.dtype(np.float64), 3, 4, 0.5, 4, seed=2)
    g = gpu_run(w, init=init, variant=variant, sampler=SLICE)
    r = ref_run(w, init=init, sampler=SLICE)
    assert (g[1] == 1).all() and np.array_equal(g[1], r[1]) and np.array_equal(g[2], r[2]) and np.array_equal(g[0], r[0])


def test_slice_sampler_dense_gaussian_config2():
    w = W.make(2, n_chains=24, n_iters=20)
    assert_parity(gpu_run(w, sampler=SLICE), ref_run(w, sampler=SLICE), F64_TOL, label="config 2, slice")
    assert_parity(gpu_run(w, sampler=SLICE, leaf_steps=4), ref_run(w, sampler=SLICE, leaf_steps=4), F64_TOL,
                  label="config 2, slice, 4 steps per leaf (the paper's setting)")


@pytest.mark.parametrize("n_data,dim", [(5, 2), (65, 17), (1000, 25), (129, 32)])
def test_slice_sampler_logreg_tile_and_wave_kernels(n_data, dim):
    w = W.small_logreg(n_data, dim, seed=100 + n_data)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 21, 12, 0.15 / np.sqrt(max(n_data, 1) / 10), 7
    B = N()
    r = ref_run(w, sampler=SLICE)
    for variant in (B.NUTS_VARIANT_TILE, B.NUTS_VARIANT_WAVE):
        g = gpu_run(w, variant=variant, sampler=SLICE)
        assert g[3]["variant"] == variant and g[3]["leaf_slots_useful"] == g[2].sum()
        assert_parity(g, r, F64_TOL, label=f"{w.name} variant {variant}, slice")
    r = ref_run(w, sampler=SLICE, leaf_steps=2)
    g = gpu_run(w, variant=B.NUTS_VARIANT_TILE, sampler=SLICE, leaf_steps=2, schedule=B.NUTS_SCHEDULE_TRAJECTORY)
    assert_parity(g, r, F64_TOL, label=f"{w.name} tile, slice, 2 steps per leaf, trajectory schedule")


def test_slice_sampler_config3_tile_kernel_at_full_chain_count():
    w = W.make(3, n_iters=30)
    B = N()
    g = gpu_run(w, variant=B.NUTS_VARIANT_TILE, sampler=SLICE)
    check_invariants(w, g[1], g[2])
    ids = np.concatenate([np.arange(8), np.random.default_rng(3).choice(4096, 32, replace=False), [4095]])
    assert_parity(g, ref_run(w, chain_ids=ids, sampler=SLICE), F64_TOL, cols=ids, label="config 3, slice")


def test_slice_sampler_tile_kernel_divergences_and_deep_trees():
    B = N()
    w = W.small_logreg(50, 4, seed=6)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 20, 20, 0.6, 6
    init = np.random.default_rng(1).standard_normal((20, 4)) * 5
    r = ref_run(w, init=init, sampler=SLICE)
    assert (r[2] != 2 ** r[1].astype(np.int64) - 1).sum() > 5
    assert_parity(gpu_run(w, variant=B.NUTS_VARIANT_TILE, init=init, sampler=SLICE), r, F64_TOL, label="tile divergent, slice")
    w = W.small_logreg(30, 3, seed=4)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 18, 2, 0.0005, 12
    r = ref_run(w, sampler=SLICE)
    assert r[1].max() == 12
    assert_parity(gpu_run(w, variant=B.NUTS_VARIANT_TILE, sampler=SLICE), r, F64_TOL, label="tile depth 12, slice")


def test_slice_sampler_logreg_f32_chip_kernel_and_bad_argument():
    w = W.small_logreg(1000, 33, seed=1200, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 40, 6, 0.015, 6
    B = N()
    g = gpu_run(w, variant=B.NUTS_VARIANT_GRID, sampler=SLICE)
    assert_chip(g[3])
    f32_parity(g, ref_run(w, sampler=SLICE))
    with pytest.raises(B.NutsError):
        B.nuts_sample(gpu_target(w), 2, 2, 0.1, 3, 1, sampler=2)


# ------------------------------------------------------------------ dense-Gaussian register kernel (matrix in LDS)

DENSE = 5


@pytest.mark.parametrize("dim", [1, 2, 3, 63, 64, 65, 100, 127, 128])
def test_dense_register_kernel_ragged_dimensions(dim):
    w = W.Workload(f"dense_d{dim}", W.GAUSS_DENSE, dim, np.dtype(np.float64), 7, 10, 0.2, 7, seed=6,
                   precision=W.random_spd_precision(dim, 3))
    g = gpu_run(w, variant=DENSE)
    assert g[3]["variant"] == DENSE and g[3]["leaf_slots_useful"] == g[2].sum() and g[3]["extra_grad_evals"] == 7
    assert_parity(g, ref_run(w), F64_TOL, label=w.name)
    auto = gpu_run(w)
    assert auto[3]["variant"] == DENSE
    for a, b in zip(g[:3], auto[:3]):
        assert np.array_equal(a, b)


def test_dense_register_kernel_config2_full_chain_count_and_queueing():
    w = W.make(2, n_iters=50)
    g = gpu_run(w)
    assert g[3]["variant"] == DENSE
    check_invariants(w, g[1], g[2])
    ids = np.array([0, 1, 2, 3, 500, 777, 1022, 1023])
    assert_parity(g, ref_run(w, chain_ids=ids), F64_TOL, cols=ids, label="config 2, dense kernel")
    w = W.make(2, n_chains=5000, n_iters=2)          # more chains than resident slots: the queue refills them
    g = gpu_run(w)
    ids = np.array([0, 1023, 1024, 2047, 2048, 4999])
    assert_parity(g, ref_run(w, chain_ids=ids), F64_TOL, cols=ids, label="config 2, queued chains")


def test_dense_register_kernel_options_and_limits():
    B = N()
    w = W.make(2, n_chains=24, n_iters=12)
    for kw in (dict(leaf_steps=4), dict(sampler=SLICE), dict(sampler=SLICE, leaf_steps=2)):
        g = gpu_run(w, variant=DENSE, **kw)
        assert_parity(g, ref_run(w, **kw), F64_TOL, label=f"config 2 dense kernel {kw}")
    free, sync = both_schedules(w, DENSE)
    init = np.random.default_rng(3).standard_normal((24, w.dim)) * 10      # far out, near the stability limit
    w.step_size = 0.44
    g = gpu_run(w, variant=DENSE, init=init)
    r = ref_run(w, init=init)
    assert (r[2] != 2 ** r[1].astype(np.int64) - 1).sum() > 5
    assert_parity(g, r, F64_TOL, label="config 2 dense kernel, divergent")
    # much further out: leaves land thousands below the starting energy, and the unit of the weights moves
    init = np.random.default_rng(4).standard_normal((24, w.dim)) * 60
    w.step_size = 0.3
    assert_parity(gpu_run(w, variant=DENSE, init=init), ref_run(w, init=init), F64_TOL, label="config 2 dense kernel, far start")
    big = W.Workload("dense_d129", W.GAUSS_DENSE, 129, np.dtype(np.float64), 3, 2, 0.2, 4, seed=6,
                     precision=W.random_spd_precision(129, 3))
    with pytest.raises(B.NutsError):
        gpu_run(big, variant=DENSE)
    assert gpu_run(big)[3]["variant"] == B.NUTS_VARIANT_WAVE


def test_dense_register_kernel_f32():
    P = W.random_spd_precision(70, 5).astype(np.float32)
    w = W.Workload("dense32", W.GAUSS_DENSE, 70, np.dtype(np.float32), 12, 6, 0.2, 6, seed=9, precision=P)
    g = gpu_run(w, variant=DENSE)
    assert g[3]["variant"] == DENSE
    f32_parity(g, ref_run(w))


# ------------------------------------------------------------------ quad kernel (four chains per wavefront, P theta on MFMA blocks)

QUAD = 6


@pytest.mark.parametrize("dim,n_chains", [(1, 1), (2, 3), (3, 4), (15, 5), (16, 16), (17, 21), (63, 33), (64, 7), (65, 64),
                                           (100, 37), (127, 9), (128, 70)])
def test_quad_kernel_ragged_dimensions_and_chain_counts(dim, n_chains):
    w = W.Workload(f"quad_d{dim}", W.GAUSS_DENSE, dim, np.dtype(np.float64), n_chains, 10, 0.2, 7, seed=6 + dim,
                   precision=W.random_spd_precision(dim, 3))
    g = gpu_run(w, variant=QUAD)
    assert g[3]["variant"] == QUAD and g[3]["leaf_slots_useful"] == g[2].sum() and g[3]["extra_grad_evals"] == n_chains
    r = ref_run(w)
    assert r[2].max() >= 3
    assert_parity(g, r, F64_TOL, label=w.name)
    dense = gpu_run(w, variant=DENSE)            # the two kernels sum in different orders: same integers, states to rounding
    assert np.array_equal(dense[1], g[1]) and np.array_equal(dense[2], g[2])


def test_quad_kernel_random_spd_d100_many_chains_queueing_and_independence():
    """The case the kernel is for: a correlated Gaussian whose precision is not banded, more chains than resident
    slots (256 compute units x 16), chosen automatically."""
    w = W.Workload("quad_spd_d100", W.GAUSS_DENSE, 100, np.dtype(np.float64), 6000, 4, 0.15, 8, seed=21,
                   precision=W.random_spd_precision(100, 7))
    tgt = gpu_target(w)
    g = gpu_run(w, tgt=tgt)
    assert g[3]["variant"] == QUAD
    check_invariants(w, g[1], g[2])
    assert np.isfinite(g[0]).all()
    ids = np.array([0, 1, 2, 3, 4, 15, 16, 4095, 4096, 4097, 5999])
    assert_parity(g, ref_run(w, chain_ids=ids), F64_TOL, cols=ids, label="quad, queued chains")
    st = g[3]
    assert st["leaf_slots_useful"] == g[2].sum() and st["leaf_slots_issued"] >= st["leaf_slots_useful"] + 6000
    small = gpu_run(w, variant=QUAD, tgt=tgt, n_chains=5)
    off = gpu_run(w, variant=QUAD, tgt=tgt, n_chains=33, first_chain=3000)
    again = gpu_run(w, tgt=tgt)
    for k in range(3):
        assert np.array_equal(g[k][:, :5], small[k])          # a chain's results do not depend on the batch it runs in
        assert np.array_equal(g[k][:, 3000:3033], off[k])
        assert np.array_equal(g[k], again[k])
    few = gpu_run(w, tgt=tgt, n_chains=100)                    # few chains: one chain per wavefront spreads them better
    assert few[3]["variant"] == DENSE


def test_quad_kernel_options_deep_trees_and_divergences():
    B = N()
    w = W.Workload("quad_opts", W.GAUSS_DENSE, 40, np.dtype(np.float64), 23, 8, 0.25, 7, seed=5,
                   precision=W.random_spd_precision(40, 2))
    for kw in (dict(leaf_steps=4), dict(sampler=SLICE), dict(sampler=SLICE, leaf_steps=2)):
        assert_parity(gpu_run(w, variant=QUAD, **kw), ref_run(w, **kw), F64_TOL, label=f"quad {kw}")
    both_schedules(w, QUAD)
    both_schedules(w, QUAD, sampler=SLICE, leaf_steps=3)
    # deep trees up to the depth limit of the kernel
    w.step_size, w.max_tree_depth, w.n_iters, w.n_chains = 0.004, 10, 2, 6
    r = ref_run(w)
    assert r[1].max() == 10 and r[2].max() == 1023
    assert_parity(gpu_run(w, variant=QUAD), r, F64_TOL, label="quad deep")
    w.max_tree_depth, w.n_iters = 12, 1
    assert_parity(gpu_run(w, variant=QUAD), ref_run(w), F64_TOL, label="quad depth 12")
    w.max_tree_depth = 13
    with pytest.raises(B.NutsError):
        gpu_run(w, variant=QUAD)
    # far out and near the stability limit: divergent leaves, early exits, non-finite states
    w.step_size, w.max_tree_depth, w.n_iters, w.n_chains = 0.9, 6, 12, 20
    init = np.random.default_rng(3).standard_normal((20, w.dim)) * 10
    init[3] = 1e200
    init[7] = np.inf
    g = gpu_run(w, variant=QUAD, init=init)
    r = ref_run(w, init=init)
    assert (r[2] != 2 ** r[1].astype(np.int64) - 1).sum() > 5
    assert np.array_equal(np.isfinite(g[0]), np.isfinite(r[0]))
    assert np.array_equal(g[1], r[1]) and np.array_equal(g[2], r[2])
    fin = np.isfinite(r[0]).all(axis=(0, 2))
    assert state_error(g[0][:, fin], r[0][:, fin]) < F64_TOL
    f32 = W.Workload("quad_f32", W.GAUSS_DENSE, 8, np.dtype(np.float32), 4, 2, 0.2, 4, seed=1,
                     precision=W.random_spd_precision(8, 1).astype(np.float32))
    with pytest.raises(B.NutsError):
        gpu_run(f32, variant=QUAD)


# ------------------------------------------------------------------ the launches bench.py times, at full size

def full_size_run(cfg, **kw):
    """The exact launch of the benchmark (all chains, all iterations); only slices leave the GPU."""
    import torch
    B = N()
    w = W.make(cfg)
    tgt = gpu_target(w)
    s, d, n = B.nuts_sample(tgt, w.n_chains, w.n_iters, w.step_size, w.max_tree_depth, w.seed, **kw)
    torch.cuda.synchronize()
    return w, s, d, n, B.nuts_get_stats(tgt)


def test_config3_full_size_launch_first_50_iterations_and_invariants_everywhere():
    import torch
    w, s, d, n, st = full_size_run(3)
    assert st["variant"] == N().NUTS_VARIANT_TILE and st["leaf_slots_useful"] == int(n.sum().item())
    assert st["occupancy"] > 0.9
    dd, nn = d.to(torch.int64), n.to(torch.int64)
    assert bool(((dd >= 1) & (dd <= w.max_tree_depth) & (nn >= 2 ** (dd - 1)) & (nn <= 2 ** dd - 1)).all())
    assert bool(torch.isfinite(s).all())
    ids = np.concatenate([np.arange(4), np.random.default_rng(11).choice(4096, 20, replace=False), [4095]])
    r = ref_run(w, chain_ids=ids, n_iters=50)
    t = torch.as_tensor(ids).cuda()
    g = (s[:50][:, t].cpu().numpy(), d[:50][:, t].cpu().numpy(), n[:50][:, t].cpu().numpy())
    assert_parity(g, r, F64_TOL, label="config 3 at full size, first 50 iterations")
    # the sample itself: posterior means of all chains agree across two halves of the chains
    late = s[200:]
    a, b = late[:, :2048].mean(dim=(0, 1)), late[:, 2048:].mean(dim=(0, 1))
    assert float((a - b).abs().max()) < 0.02


def test_config2_full_size_launch_first_50_iterations():
    import torch
    w, s, d, n, st = full_size_run(2)
    assert st["variant"] == DENSE
    ids = np.array([0, 1, 511, 512, 1023])
    r = ref_run(w, chain_ids=ids, n_iters=50)
    t = torch.as_tensor(ids).cuda()
    g = (s[:50][:, t].cpu().numpy(), d[:50][:, t].cpu().numpy(), n[:50][:, t].cpu().numpy())
    assert_parity(g, r, F64_TOL, label="config 2 at full size, first 50 iterations")
    x = s[300:].reshape(-1, w.dim)
    cov = torch.cov(x.T).cpu().numpy()
    want = 0.9 ** np.abs(np.subtract.outer(np.arange(w.dim), np.arange(w.dim)))
    assert np.abs(cov - want).max() < 0.08 and float(x.mean(dim=0).abs().max()) < 0.05


def test_config4_full_size_launch_first_10_iterations_binary32():
    import torch
    w, s, d, n, st = full_size_run(4)
    assert st["variant"] == N().NUTS_VARIANT_GRID
    ids = np.arange(8)
    r = ref_run(w, chain_ids=ids, n_iters=10)
    g = (s[:10, :8].cpu().numpy(), d[:10, :8].cpu().numpy(), n[:10, :8].cpu().numpy())
    f32_parity(g, r)
    assert bool(torch.isfinite(s).all())


def test_config5_full_size_launch_first_20_iterations_binary32_and_invariants_everywhere():
    """The launch bench.py times on configuration 5: 16384 chains x 500 iterations, chains beyond the resident slots
    taken from the queue.  Sampled chains against the oracle over their first 20 iterations, per coordinate (the
    scales span four decades); structural invariants and finiteness over everything; the sample itself against the
    target's standard deviations."""
    import torch
    w, s, d, n, st = full_size_run(5)
    assert st["variant"] == N().NUTS_VARIANT_ELEM and st["leaf_slots_useful"] == int(n.sum().item())
    dd, nn = d.to(torch.int64), n.to(torch.int64)
    assert bool(((dd >= 1) & (dd <= w.max_tree_depth) & (nn >= 2 ** (dd - 1)) & (nn <= 2 ** dd - 1)).all())
    assert bool(torch.isfinite(s).all())
    ids = np.concatenate([np.arange(4), np.random.default_rng(5).choice(16384, 27, replace=False), [16383]])
    r = ref_run(w, chain_ids=ids, n_iters=20)
    t = torch.as_tensor(ids).cuda()
    g = (s[:20][:, t].cpu().numpy(), d[:20][:, t].cpu().numpy(), n[:20][:, t].cpu().numpy())
    f32_parity(g, r)
    # late iterations, a slice of the chains: every coordinate's spread is its sigma (trajectories of at most 1023 steps
    # of 0.01 do not cross the widest coordinates in one iteration, so those are still narrower than their sigma)
    x = s[300::20, ::8].reshape(-1, w.dim).to(torch.float64)
    ratio = (x.std(dim=0).cpu().numpy() / w.scales.astype(np.float64))
    narrow = w.scales < 1.0
    assert np.abs(ratio[narrow] - 1.0).max() < 0.1 and (ratio <= 1.1).all()
    del s, x


# ------------------------------------------------------------------ option matrix: every kernel x sampler x leaf size x schedule

def _matrix_cases():
    rng = np.random.default_rng(2024)
    cases = []
    for variant, kind in [(1, "std"), (3, "std"), (1, "diag"), (3, "diag"), (1, "dense"), (5, "dense"), (1, "logreg"),
                          (2, "logreg"), (4, "logreg32")]:
        for rep in range(4):
            cases.append((variant, kind, int(rng.integers(0, 2)), int(rng.choice([1, 2, 3, 5])), int(rng.integers(0, 2)),
                          int(rng.integers(1, 40)), int(rng.integers(1, 30)), int(rng.integers(0, 10**6))))
    return cases


@pytest.mark.parametrize("variant,kind,sampler,k,schedule,dim,n_chains,seed", _matrix_cases())
def test_option_matrix(variant, kind, sampler, k, schedule, dim, n_chains, seed):
    rng = np.random.default_rng(seed)
    n_iters, depth = 6, 6
    if kind == "std":
        w = W.Workload("m_std", W.STD_NORMAL, dim, np.dtype(np.float64), n_chains, n_iters, 0.5 / k, depth, seed=seed)
    elif kind == "diag":
        w = W.Workload("m_diag", W.GAUSS_DIAG, dim, np.dtype(np.float64), n_chains, n_iters, 0.1 / k, depth, seed=seed,
                       scales=10.0 ** rng.uniform(-0.5, 0.5, dim))
    elif kind == "dense":
        w = W.Workload("m_dense", W.GAUSS_DENSE, dim, np.dtype(np.float64), n_chains, n_iters, 0.3 / k, depth, seed=seed,
                       precision=W.random_spd_precision(dim, seed % 7))
    else:
        dim = min(dim, 32)
        n_data = int(rng.integers(1, 300))
        w = W.small_logreg(n_data, dim, seed=seed, dtype=np.float32 if kind == "logreg32" else np.float64)
        w.n_chains, w.n_iters, w.max_tree_depth = n_chains, n_iters, depth
        w.step_size = 0.3 / k / np.sqrt(max(n_data, 10) / 10)
        w.seed = seed
    g = gpu_run(w, variant=variant, sampler=sampler, leaf_steps=k, schedule=schedule)
    r = ref_run(w, sampler=sampler, leaf_steps=k)
    assert g[3]["variant"] == variant
    if kind == "logreg32":
        f32_parity(g, r)
    else:
        assert_parity(g, r, F64_TOL, label=f"{kind} v{variant} sampler={sampler} k={k} schedule={schedule} d={w.dim}")


def banded_spd(dim, half, seed):
    """A symmetric positive definite matrix that is exactly zero beyond `half` off-diagonals."""
    rng = np.random.default_rng(seed)
    P = np.zeros((dim, dim))
    for k in range(1, half + 1):
        v = rng.uniform(-0.4, 0.4, dim - k) if dim > k else np.zeros(0)
        P += np.diag(v, k) + np.diag(v, -k)
    return P + np.diag(np.abs(P).sum(axis=1) + rng.uniform(0.5, 2.0, dim))


@pytest.mark.parametrize("dim,half", [(1, 0), (2, 1), (9, 4), (100, 1), (100, 4), (128, 3), (127, 5), (40, 39)])
def test_dense_register_kernel_banded_and_nearly_banded_matrices(dim, half):
    """Up to four off-diagonals the kernel keeps the band in registers; beyond that it falls back to the
    matrix in LDS.  Both must match the oracle's dense sums."""
    half = min(half, dim - 1)
    w = W.Workload(f"band_d{dim}_h{half}", W.GAUSS_DENSE, dim, np.dtype(np.float64), 9, 10, 0.25, 7, seed=dim + half,
                   precision=banded_spd(dim, half, seed=dim))
    g = gpu_run(w, variant=DENSE)
    assert g[3]["variant"] == DENSE
    r = ref_run(w)
    assert r[2].max() >= 3
    assert_parity(g, r, F64_TOL, label=w.name)
    wave = gpu_run(w, variant=1)
    assert np.array_equal(wave[1], g[1]) and np.array_equal(wave[2], g[2])


def test_dense_register_kernel_banded_f32_and_options():
    P = banded_spd(60, 2, seed=3).astype(np.float32)
    w = W.Workload("band32", W.GAUSS_DENSE, 60, np.dtype(np.float32), 12, 6, 0.2, 6, seed=9, precision=P)
    f32_parity(gpu_run(w, variant=DENSE), ref_run(w))
    w = W.make(2, n_chains=24, n_iters=12)        # the AR(1) precision of configuration 2 is tridiagonal
    for kw in (dict(leaf_steps=4), dict(sampler=SLICE), dict(sampler=SLICE, leaf_steps=2)):
        assert_parity(gpu_run(w, variant=DENSE, **kw), ref_run(w, **kw), F64_TOL, label=f"banded {kw}")
    both_schedules(w, DENSE)


# ------------------------------------------------------------------ wide tile kernel (up to 128 features, both dtypes, 16 or 4 chains in lock step)

def wide_workload(n_data, dim, dtype, n_chains):
    w = W.small_logreg(n_data, dim, seed=900 + n_data + dim, dtype=dtype)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = n_chains, 6, 0.15 / np.sqrt(max(n_data, 1) / 10), 6
    return w


# feature counts at the edges of the tiles of 16, of the k-steps of 4 (also with the constant column outside the first
# GEMM: d = 1 mod 4) and of the components per lane; row counts below, at and beyond a tile and a round of 8 tiles
@pytest.mark.parametrize("n_data,dim", [(1, 33), (15, 48), (16, 49), (129, 63), (128, 64), (300, 65), (77, 80), (145, 81), (40, 96),
                                        (131, 97), (64, 112), (17, 113), (129, 128), (9000, 34)])
def test_wide_kernel_f64_both_forms_match_the_oracle_and_each_other(n_data, dim):
    B = N()
    w = wide_workload(n_data, dim, np.float64, 9 if n_data < 9000 else 3)
    tgt = gpu_target(w)
    few = gpu_run(w, tgt=tgt)                              # four chains per workgroup
    assert few[3]["variant"] == B.NUTS_VARIANT_TILE and few[3]["leaf_slots_useful"] == few[2].sum()
    assert_parity(few, ref_run(w), F64_TOL, label=w.name)
    many = gpu_run(w, tgt=tgt, n_chains=2100, n_iters=2)    # sixteen
    for k in range(3):                                      # the same bits whichever form computes a chain
        assert np.array_equal(many[k][:, :w.n_chains], few[k][:2])


@pytest.mark.parametrize("n_data,dim", [(1, 1), (50, 5), (700, 17), (131, 32), (200, 33), (129, 100), (120, 128)])
def test_wide_kernel_f32_small_data_sets_keep_the_sums_of_the_wave_kernel(n_data, dim):
    B = N()
    w = wide_workload(n_data, dim, np.float32, 13)
    tgt = gpu_target(w)
    g = gpu_run(w, tgt=tgt)
    assert g[3]["variant"] == B.NUTS_VARIANT_TILE
    f32_parity(g, ref_run(w))
    slice4 = gpu_run(w, tgt=tgt, sampler=1, leaf_steps=4, schedule=1)
    f32_parity(slice4, ref_run(w, sampler=1, leaf_steps=4))
    many = gpu_run(w, tgt=tgt, n_chains=2100, n_iters=2)
    for k in range(3):
        assert np.array_equal(many[k][:, :13], g[k][:2])


@pytest.mark.parametrize("n_chains", [1, 5, 1023])
def test_tile_kernel_four_chain_form_deep_trees_divergences_and_options(n_chains):
    """Up to 4 chains per compute unit the tile variant steps 4 chains per workgroup: the same bits as 16 per workgroup."""
    w = W.small_logreg(50, 5, seed=6)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = n_chains, 8, 0.5, 7
    init = np.random.default_rng(1).standard_normal((n_chains, 5)) * 8
    tgt = gpu_target(w)
    r = ref_run(w, init=init)
    g = gpu_run(w, tgt=tgt, init=init)
    assert_parity(g, r, F64_TOL, label="four chains per workgroup")
    assert_parity(gpu_run(w, tgt=tgt, init=init, sampler=1, leaf_steps=3, schedule=1), ref_run(w, init=init, sampler=1, leaf_steps=3),
                  F64_TOL, label="four chains per workgroup, slice")
    wide = gpu_run(w, tgt=tgt, n_chains=2100, n_iters=3)
    few = gpu_run(w, tgt=tgt, n_iters=3)
    for k in range(3):
        assert np.array_equal(wide[k][:, :n_chains], few[k])


# ------------------------------------------------------------------ block kernel (dense Gaussian, 128 < d <= 512, matrix streamed from L2)

# dimensions at the edges of the row groups of 16, of the quarters of 32 columns (odd and even counts of column pairs per
# quarter) and of the components per lane; chain counts with idle slots and with more chains than a workgroup takes
@pytest.mark.parametrize("dim,dtype,n_chains", [(129, np.float64, 1), (144, np.float64, 5), (159, np.float32, 9), (161, np.float64, 4),
                                                (255, np.float64, 6), (256, np.float32, 3), (257, np.float64, 5), (320, np.float32, 5),
                                                (384, np.float64, 3), (385, np.float64, 3), (512, np.float32, 2), (512, np.float64, 2)])
def test_block_kernel_ragged_dimensions_and_chain_counts(dim, dtype, n_chains):
    P = W.random_spd_precision(dim, 3).astype(dtype)
    w = W.Workload(f"block_d{dim}", W.GAUSS_DENSE, dim, np.dtype(dtype), n_chains, 5, 0.2, 7, seed=6 + dim, precision=P)
    tgt = gpu_target(w)
    g, r = gpu_run(w, tgt=tgt), ref_run(w)
    assert g[3]["leaf_slots_useful"] == g[2].sum() and g[3]["extra_grad_evals"] == n_chains
    assert g[3]["rounds"] < g[3]["leaf_slots_useful"] or n_chains == 1         # chains share rounds
    check = (lambda a, b, label: assert_parity(a, b, F64_TOL, label=label)) if dtype is np.float64 else (lambda a, b, label: f32_parity(a, b))
    check(g, r, w.name)
    kw = dict(sampler=SLICE, leaf_steps=3, schedule=1)
    check(gpu_run(w, tgt=tgt, **kw), ref_run(w, sampler=SLICE, leaf_steps=3), f"{w.name} slice")


@pytest.mark.parametrize("dim,dtype", [(130, np.float64), (250, np.float32), (300, np.float64)])
def test_block_kernel_both_forms_give_the_same_bits_and_chains_are_independent(dim, dtype):
    w = W.Workload(f"block_many_d{dim}", W.GAUSS_DENSE, dim, np.dtype(dtype), 2500, 2, 0.2, 6, seed=3,
                   precision=W.random_spd_precision(dim, 5).astype(dtype))
    tgt = gpu_target(w)
    many = gpu_run(w, tgt=tgt)                                  # eight chains per workgroup, some from the queue
    few = gpu_run(w, tgt=tgt, n_chains=9, first_chain=2045)      # four
    again = gpu_run(w, tgt=tgt)
    for k in range(3):
        assert np.array_equal(many[k][:, 2045:2054], few[k]) and np.array_equal(many[k], again[k])


def test_block_kernel_deep_trees_divergences_and_nonfinite_starts():
    w = W.Workload("block_far", W.GAUSS_DENSE, 140, np.dtype(np.float64), 12, 6, 0.9, 6, seed=4,
                   precision=W.random_spd_precision(140, 3))
    init = np.random.default_rng(3).standard_normal((12, 140)) * 10
    init[3] = 1e200
    init[7] = np.inf
    g, r = gpu_run(w, init=init), ref_run(w, init=init)
    assert np.array_equal(np.isfinite(g[0]), np.isfinite(r[0]))
    assert np.array_equal(g[1], r[1]) and np.array_equal(g[2], r[2])
    fin = np.isfinite(r[0]).all(axis=(0, 2))
    assert state_error(g[0][:, fin], r[0][:, fin]) < F64_TOL
    w.step_size, w.max_tree_depth, w.n_iters, w.n_chains = 0.004, 10, 2, 3    # deep trees: levels beyond those in LDS
    assert_parity(gpu_run(w), ref_run(w), F64_TOL, label="block kernel, deep trees")


@pytest.mark.parametrize("dim,dtype", [(129, np.float64), (200, np.float32), (257, np.float32), (512, np.float64), (513, np.float64),
                                       (1025, np.float64), (2049, np.float32)])
def test_banded_precision_beyond_the_register_kernel(dim, dtype):
    """AUTO's kernel for banded matrices of up to 2048 dimensions against the oracle; the wave kernel, which takes nine
    entries of each row, and, with one entry off the band, all of them: the same bits."""
    P = W.ar1_precision(dim, 0.8)
    P[5, 1] = P[1, 5] = 0.05
    w = W.Workload(f"band_d{dim}", W.GAUSS_DENSE, dim, np.dtype(dtype), 5, 3, 0.1, 6, seed=8, precision=P.astype(dtype))
    off = P.copy()
    off[9, 3] = off[3, 9] = 1e-300 if dtype is np.float64 else 1e-38
    check = (lambda a, b: assert_parity(a, b, F64_TOL, label=w.name)) if dtype is np.float64 else f32_parity
    g = gpu_run(w)
    check(g, ref_run(w))
    nine = gpu_run(w, variant=N().NUTS_VARIANT_WAVE)
    kw = dict(sampler=SLICE, leaf_steps=3, schedule=1)
    s3, s3w = gpu_run(w, **kw), gpu_run(w, variant=N().NUTS_VARIANT_WAVE, **kw)
    for k in range(3):
        assert np.array_equal(g[k], nine[k]) and np.array_equal(s3[k], s3w[k])
    w.precision = off.astype(dtype)
    full = gpu_run(w, variant=N().NUTS_VARIANT_WAVE)
    for k in range(3):
        assert np.array_equal(g[k], full[k])


# ------------------------------------------------------------------ element-wise targets over the register kernel's whole range

@pytest.mark.parametrize("dim,dtype", [(129, np.float64), (256, np.float32), (513, np.float64), (1024, np.float64), (1025, np.float32),
                                       (1025, np.float64), (2048, np.float64), (2049, np.float32)])
def test_elementwise_targets_up_to_and_beyond_the_register_kernel(dim, dtype):
    """AUTO against the oracle and, bit for bit in the states, against the general wave kernel."""
    sig = (10.0 ** np.random.default_rng(dim).uniform(-1, 1, dim)).astype(dtype)
    w = W.Workload(f"elem_d{dim}", W.GAUSS_DIAG, dim, np.dtype(dtype), 6, 3, 0.02, 8, seed=19, scales=sig)
    g = gpu_run(w)
    assert g[3]["leaf_slots_useful"] == g[2].sum() and g[2].max() > 32        # deep enough for tree levels outside LDS
    if dtype is np.float64:
        assert_parity(g, ref_run(w), F64_TOL, label=w.name)
    else:
        f32_parity(g, ref_run(w))
    general = gpu_run(w, variant=N().NUTS_VARIANT_WAVE)
    for k in range(3):
        assert np.array_equal(g[k], general[k])
    kw = dict(sampler=SLICE, leaf_steps=3, schedule=1)
    for a, b in zip(gpu_run(w, **kw)[:3], gpu_run(w, variant=N().NUTS_VARIANT_WAVE, **kw)[:3]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n_chains", [128, 129, 256, 260, 700, 1100])
@pytest.mark.parametrize("n_data,dim,which", [(3000, 9, assert_chip), (12001, 17, assert_grid)])
def test_chip_and_grid_kernels_pack_the_chains_that_want_a_gradient(n_data, dim, which, n_chains):
    """Columns are handed out round by round (by the grid kernels beyond 128 chains per stream): a chain's results have the same
    bits in any company, on either schedule, whichever column its gradient was computed in."""
    B = N()
    w = W.small_logreg(n_data, dim, seed=77, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = n_chains, 4, 1.1 / np.sqrt(n_data), 7 if which is assert_chip else 5
    tgt = gpu_target(w)
    g = gpu_run(w, tgt=tgt, variant=B.NUTS_VARIANT_GRID)
    which(g[3])
    assert g[3]["leaf_slots_issued"] >= g[3]["leaf_slots_useful"] + g[3]["extra_grad_evals"]
    assert len(set(g[2].sum(axis=0))) > 3                       # trajectories of different lengths: idle slots in between
    sync = gpu_run(w, tgt=tgt, variant=B.NUTS_VARIANT_GRID, schedule=1)
    few = gpu_run(w, tgt=tgt, variant=B.NUTS_VARIANT_GRID, n_chains=6, first_chain=n_chains - 6)
    for k in range(3):
        assert np.array_equal(g[k], sync[k])
        assert np.array_equal(g[k][:, n_chains - 6:], few[k])
    pick = np.arange(4)
    f32_parity([x[:, :4] for x in g[:3]], ref_run(w, chain_ids=pick))


def test_more_than_a_million_rows_stay_on_the_tile_variant():
    """The tile variant takes binary64 data sets of up to four million rows (dim <= 32), and AUTO leaves none of them to the
    general wave kernel; nuts_sample_static takes them too (the wave kernel would need 8 bytes per row and chain slot)."""
    import torch
    B = N()
    n, d = 1_000_001, 3
    rng = np.random.default_rng(11)
    X = np.concatenate([rng.standard_normal((n, d - 1)), np.ones((n, 1))], axis=1)
    y = (rng.random(n) < 1.0 / (1.0 + np.exp(-X @ np.array([0.4, -0.3, 0.1])))).astype(np.float64)
    w = W.Workload("logreg_1000001x3", W.LOGREG, d, np.dtype(np.float64), 70, 2, 5e-4, 3, seed=12, X=X, y=y, prior_scale=1.0)
    tgt = gpu_target(w)
    g = gpu_run(w, tgt=tgt)
    assert g[3]["variant"] == B.NUTS_VARIANT_TILE
    asked = gpu_run(w, tgt=tgt, variant=B.NUTS_VARIANT_TILE)
    many = gpu_run(w, tgt=tgt, n_chains=2100, n_iters=1)         # sixteen chains per workgroup
    static = B.nuts_sample(tgt, w.n_chains, w.n_iters, w.step_size, w.max_tree_depth, w.seed, static_scratch=True)
    torch.cuda.synchronize()
    for k in range(3):
        assert np.array_equal(g[k], asked[k]) and np.array_equal(g[k], static[k].cpu().numpy())
        assert np.array_equal(g[k][0], many[k][0, :w.n_chains])
    assert_parity([x[:, :2] for x in g[:3]], ref_run(w, chain_ids=np.arange(2)), F64_TOL, label=w.name)


# Rounding made visible: logits of 1e12 and a step size to match.  The likelihood is linear as far as a trajectory reaches,
# so its energy is constant up to the rounding of sums of 1e14, which is of the order of 0.01 and decides selections in
# some of the thousands of trees.  Any difference in how the forms add up a log-likelihood shows.
@pytest.mark.parametrize("n_data,dim", [(300, 3), (131, 17), (300, 25), (1100, 32), (9000, 5), (300, 40), (145, 100)])
def test_chains_have_the_same_bits_in_either_lock_step_form_where_rounding_decides(n_data, dim):
    rng = np.random.default_rng(dim)
    X = 1e12 * rng.standard_normal((n_data, dim))
    if dim == 25:
        X[:, 7] = 1e12                                            # a constant column that stays out of the first GEMM
    y = (rng.random(n_data) < 0.5).astype(np.float64)
    w = W.Workload("rounding", W.LOGREG, dim, np.dtype(np.float64), 1000, 6, 2e-13 * (300 / n_data) ** 0.5, 5, seed=4, X=X, y=y, prior_scale=1.0)
    tgt = gpu_target(w)
    few = gpu_run(w, tgt=tgt)                                     # four chains per workgroup
    many = gpu_run(w, tgt=tgt, n_chains=4096)                     # sixteen
    assert len(np.unique(few[2])) > 3
    for k in range(3):
        differ = (few[k] != many[k][:, :w.n_chains])
        assert differ.sum() == 0, f"{differ.sum()} of {differ.size} values differ"


# One pass of the generator makes the momenta of 64 / n iterations (n: pairs of components, up to a power of two): dimensions at the edges of
# n, iterations beyond one pass.
@pytest.mark.parametrize("dim,dtype", [(1, np.float64), (2, np.float64), (3, np.float32), (4, np.float64), (5, np.float64), (9, np.float32), (17, np.float64),
                                       (32, np.float64), (33, np.float64), (64, np.float32), (65, np.float64), (128, np.float64)])
def test_momenta_made_for_several_iterations_at_once(dim, dtype):
    sig = 10.0 ** np.linspace(-0.3, 0.3, dim)
    w = W.Workload("several", W.GAUSS_DIAG, dim, np.dtype(dtype), 5, 131, 0.3, 4, seed=23, scales=sig)
    g = gpu_run(w)
    assert_parity(g, ref_run(w), F64_TOL if dtype == np.float64 else F32_TOL, exact_ints=dtype == np.float64, label=f"several {dim}")
    for x, y in zip(gpu_run(w, schedule=1)[:3], g[:3]):           # a launch per iteration: a pass each
        assert np.array_equal(x, y)


def workspace_of(tgt, most=0):
    """Bytes of workspace and refused allocations so far; from now on those of more than `most` bytes are refused (0: none)."""
    import ctypes as C
    size, refusals = C.c_uint64(), C.c_int()
    N()._check(N().lib().nuts_debug_workspace(tgt.handle, C.c_uint64(most), C.byref(size), C.byref(refusals)))
    return size.value, refusals.value


def counts_of(tgt):
    """Of the last call: pairs of workgroups that met, pairs of which one went on alone, chains handed over to another slot."""
    import ctypes as C
    c = [C.c_uint64() for _ in range(3)]
    N()._check(N().lib().nuts_debug_counts(tgt.handle, *[C.byref(x) for x in c]))
    return tuple(x.value for x in c)


# Every instance that takes turns (components of a lane: the edges of each), a turn after every iteration that leaves another chain waiting;
# chains that all take turns and (more than eight for a slot) chains of which only the last do.
@pytest.mark.parametrize("kind,dim,dtype,chains,iters", [
    (W.GAUSS_DIAG, 3, np.float64, 8001, 9), (W.GAUSS_DIAG, 128, np.float32, 30011, 5), (W.GAUSS_DIAG, 129, np.float64, 3001, 6), (W.GAUSS_DIAG, 256, np.float32, 4099, 6),
    (W.GAUSS_DIAG, 257, np.float32, 3001, 6), (W.GAUSS_DIAG, 500, np.float64, 2203, 6), (W.GAUSS_DIAG, 777, np.float64, 1031, 5), (W.GAUSS_DIAG, 1000, np.float32, 2051, 5),
    (W.GAUSS_DIAG, 1025, np.float32, 1031, 5), ("ar1", 100, np.float64, 2051, 7), ("ar1", 7, np.float64, 20011, 5), ("ar1", 127, np.float32, 2051, 7), ("spd", 64, np.float64, 1301, 7), ("spd", 101, np.float32, 2051, 7)])
def test_chains_are_handed_over_and_keep_their_bits(kind, dim, dtype, chains, iters):
    import ctypes as C
    w = W.Workload("turns", kind if kind == W.GAUSS_DIAG else W.GAUSS_DENSE, dim, np.dtype(dtype), chains, iters, 0.05, 9, seed=29)
    if kind != W.GAUSS_DIAG:
        w.precision = W.ar1_precision(dim, 0.8) if kind == "ar1" else W.random_spd_precision(dim, 3)
    else:
        w.scales = 10.0 ** (-1.0 + 2.0 * np.random.default_rng(dim).random(dim))
    tgt = gpu_target(w)
    N()._check(N().lib().nuts_debug_turns(tgt.handle, C.c_int(0)))
    turns = gpu_run(w, tgt=tgt)
    slots = turns[3]["grid_blocks"] * 4
    assert slots < chains and counts_of(tgt)[2] > slots
    kept = gpu_run(w, tgt=tgt, schedule=1)                        # a launch per iteration
    assert counts_of(tgt)[2] == 0
    for k in range(3):
        assert np.array_equal(turns[k], kept[k])
    assert turns[3]["leaf_slots_useful"] == turns[2].sum() and turns[3]["extra_grad_evals"] == chains


def test_which_calls_take_turns():
    import ctypes as C
    diag = dict(scales=np.ones(600))
    ar1, spd = dict(precision=W.ar1_precision(100, 0.5)), dict(precision=W.random_spd_precision(100, 3))
    for kind, dim, chains, iters, depth, want, more in [
            (W.GAUSS_DIAG, 600, 2203, 4, 9, True, diag), (W.GAUSS_DIAG, 600, 2203, 3, 10, False, diag), (W.GAUSS_DIAG, 600, 2203, 5, 8, False, diag),
            (W.GAUSS_DIAG, 600, 900, 4, 9, False, diag), (W.STD_NORMAL, 600, 2203, 4, 9, False, {}),
            (W.GAUSS_DENSE, 100, 2203, 4, 8, True, ar1), (W.GAUSS_DENSE, 100, 2203, 4, 7, False, ar1), (W.GAUSS_DENSE, 100, 2203, 4, 8, True, spd),
            (W.GAUSS_DENSE, 300, 2203, 4, 9, False, dict(precision=W.ar1_precision(300, 0.5))),
            (W.STD_NORMAL, 600, 2203, 6, 9, True, {}), (W.STD_NORMAL, 600, 2203, 5, 9, False, {}), (W.STD_NORMAL, 600, 2305, 6, 9, False, {}),
            (W.STD_NORMAL, 600, 2305, 23, 9, True, {}), (W.STD_NORMAL, 1100, 2560, 6, 9, True, {}), (W.STD_NORMAL, 1100, 2561, 6, 9, False, {}),
            (W.STD_NORMAL, 1100, 2048, 40, 9, False, {}), (W.STD_NORMAL, 60, 3200, 22, 9, False, {}), (W.STD_NORMAL, 60, 3200, 23, 9, True, {})]:
        w = W.Workload("which", kind, dim, np.dtype(np.float32), chains, iters, 0.1, depth, seed=31)
        for name, x in more.items():
            setattr(w, name, x)
        tgt = gpu_target(w)
        N()._check(N().lib().nuts_debug_turns(tgt.handle, C.c_int(0)))
        gpu_run(w, tgt=tgt)
        assert (counts_of(tgt)[2] > 0) == want, (kind, dim, chains, iters, depth)


# More chains than slots, several iterations, the steps between turns as they are: element-wise, dense and banded kernels, with vectors held in registers
# and in memory, ragged dimensions, up to eight chains per slot and more.  (That chains are handed over: the tests above.)
@pytest.mark.parametrize("kind,dim,dtype,chains,iters,eps,more", [
    (W.STD_NORMAL, 2, np.float64, 5001, 30, 0.05, {}), (W.GAUSS_DIAG, 7, np.float32, 30011, 8, 0.02, {}), (W.GAUSS_DIAG, 130, np.float64, 3100, 9, 0.02, {}),
    (W.STD_NORMAL, 500, np.float64, 2203, 12, 0.05, {}), (W.GAUSS_DIAG, 1000, np.float32, 2049, 6, 0.02, {"sampler": 1}), (W.GAUSS_DIAG, 1999, np.float32, 1027, 6, 0.02, {}),
    ("ar1", 33, np.float32, 2051, 12, 0.02, {}), ("ar1", 128, np.float64, 2050, 9, 0.05, {"leaf_steps": 4}), ("ar1", 200, np.float64, 2057, 7, 0.05, {}),
    ("ar1", 1500, np.float32, 1029, 6, 0.05, {}), ("ar1", 777, np.float64, 1029, 6, 0.05, {}), ("spd", 100, np.float64, 1031, 10, 0.05, {"variant": "NUTS_VARIANT_DENSE"})])
def test_chains_that_take_turns_have_the_bits_of_chains_that_keep_their_slot(kind, dim, dtype, chains, iters, eps, more):
    rng = np.random.default_rng(dim)
    w = W.Workload("turns", W.GAUSS_DENSE if kind in ("ar1", "spd") else kind, dim, np.dtype(dtype), chains, iters, eps, 8, seed=19)
    if kind in ("ar1", "spd"):
        w.precision = W.ar1_precision(dim, 0.8) if kind == "ar1" else W.random_spd_precision(dim, 3)
    elif kind == W.GAUSS_DIAG:
        w.scales = 10.0 ** (-1.0 + 2.0 * rng.random(dim))
    more = {k: getattr(N(), x) if k == "variant" else x for k, x in more.items()}
    tgt = gpu_target(w)
    turns = gpu_run(w, tgt=tgt, **more)
    assert turns[3]["grid_blocks"] * 4 < chains, "every chain has a slot: nothing takes turns"
    assert turns[2].sum(0).mean() > 2 * 256, "too few steps for turns"
    kept = gpu_run(w, tgt=tgt, schedule=1, **more)                # a launch per iteration: no turns
    for k in range(3):
        assert np.array_equal(turns[k], kept[k])
    assert turns[3]["leaf_slots_useful"] == turns[2].sum() and turns[3]["extra_grad_evals"] == chains
    again = gpu_run(w, tgt=tgt, n_chains=9, **more)               # a slot each
    for k in range(3):
        assert np.array_equal(again[k], turns[k][:, :9])


def test_chains_keep_their_slots_where_the_workspace_for_turns_cannot_be_had():
    w = W.Workload("turns", W.GAUSS_DIAG, 500, np.dtype(np.float64), 2203, 12, 0.05, 8, seed=19, scales=10.0 ** np.linspace(-1, 1, 500))
    tgt = gpu_target(w)
    want = gpu_run(w, tgt=tgt)
    assert want[3]["grid_blocks"] * 4 < w.n_chains
    full = workspace_of(tgt)[0]
    short = gpu_target(w)
    workspace_of(short, full - 1)
    for calls in (1, 2):
        got = gpu_run(w, tgt=short)
        size, refusals = workspace_of(short, 1)                   # (no allocation at all in the second call: what is there stays)
        assert size < full and refusals == 1                      # asked for once only
        for x, y in zip(got[:3], want[:3]):
            assert np.array_equal(x, y)


def test_awaited_iterations_need_no_workspace_for_turns():
    w = W.Workload("turns", W.GAUSS_DIAG, 500, np.dtype(np.float64), 2203, 6, 0.05, 8, seed=19, scales=10.0 ** np.linspace(-1, 1, 500))
    free, awaited = gpu_target(w), gpu_target(w)
    want, got = gpu_run(w, tgt=free), gpu_run(w, tgt=awaited, schedule=1)
    assert workspace_of(awaited)[0] == want[3]["grid_blocks"] * 4 * (4 * (w.max_tree_depth + 1) + 5) * 512 * 8 < workspace_of(free)[0]
    for x, y in zip(got[:3], want[:3]):
        assert np.array_equal(x, y)


# rows at the edges of a tile of 16, of the eight sums and of the pairs of tiles (the last of a wave's tiles alone, ragged, or with a
# ragged one beside it), on either side of 64 tiles per sum; features at the edges of the feature tiles, with and without a
# constant column, where operands are asked for a tile and half a tile ahead
@pytest.mark.parametrize("n_data,dim,dtype", [(1000, 25, np.float64), (1000, 1, np.float64), (1024, 16, np.float64), (1025, 17, np.float64), (1137, 9, np.float32),
                                              (1152, 32, np.float64), (1153, 33, np.float64), (8192, 13, np.float64), (8193, 5, np.float64), (8320, 21, np.float64),
                                              (1040, 64, np.float64), (1263, 65, np.float64), (1279, 80, np.float64), (8321, 90, np.float64), (1000, 97, np.float64),
                                              (1111, 128, np.float64), (5000, 60, np.float64), (1007, 4, np.float32)])
def test_rows_divided_between_two_workgroups_give_the_same_bits(n_data, dim, dtype):
    import ctypes as C
    w = W.small_logreg(n_data, dim, seed=dim, dtype=dtype)
    w.X[:, dim // 2] = 1.0                                        # a constant column (out of the first GEMM where dim % 4 == 1)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 11, 3, 0.7 / np.sqrt(n_data), 5
    tgt = gpu_target(w)
    pairs = gpu_run(w, tgt=tgt)
    assert pairs[3]["variant"] == N().NUTS_VARIANT_TILE and pairs[3]["grid_blocks"] == 6
    assert counts_of(tgt)[:2] == (3, 0), "pairs that did not meet have exchanged nothing"
    assert pairs[3]["leaf_slots_useful"] == pairs[2].sum() and pairs[3]["extra_grad_evals"] == w.n_chains
    whole = gpu_run(w, tgt=tgt, n_chains=1000)                    # too many chains for two workgroups of every four
    assert whole[3]["grid_blocks"] <= 250
    B = N()
    runs = [gpu_run(w, tgt=tgt, schedule=1), gpu_run(w, tgt=tgt)]
    B._check(B.lib().nuts_debug_wide_apart(tgt.handle, C.c_int(1)))   # one of the two workgroups does all
    runs.append(gpu_run(w, tgt=tgt))
    for k in range(3):
        assert np.array_equal(whole[k][:, :w.n_chains], pairs[k])
        for r in runs:
            assert np.array_equal(r[k], pairs[k])
    assert_parity(pairs, ref_run(w), F64_TOL if dtype == np.float64 else F32_TOL, exact_ints=dtype == np.float64, label="rows divided")


@pytest.mark.parametrize("n_data,dim,dtype,schedule,iters,blocks", [
    (1000, 32, np.float64, 0, 2, 6), (999, 32, np.float64, 0, 2, 3), (1000, 32, np.float64, 0, 1, 3), (1499, 5, np.float64, 1, 3, 3), (1500, 5, np.float64, 1, 3, 6),
    (1000, 33, np.float64, 1, 3, 6), (999, 33, np.float64, 0, 3, 3), (1000, 9, np.float32, 1, 3, 6)])
def test_which_calls_divide_their_rows(n_data, dim, dtype, schedule, iters, blocks):
    w = W.small_logreg(n_data, dim, seed=dim, dtype=dtype)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 11, iters, 0.02, 4
    assert gpu_run(w, schedule=schedule)[3]["grid_blocks"] == blocks


def captured_run(w, tgt, n_chains, n_iters, between, replays=3):
    """The same call captured in a graph; outputs of every replay, with `between` run after each."""
    import torch
    B, stream = N(), torch.cuda.Stream()
    tdt = torch.float64 if w.dtype == np.float64 else torch.float32
    out = (torch.empty((n_iters, n_chains, w.dim), dtype=tdt, device="cuda"), torch.empty((n_iters, n_chains), dtype=torch.int32, device="cuda"),
           torch.empty((n_iters, n_chains), dtype=torch.int32, device="cuda"))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    try:
        with torch.cuda.stream(stream):
            graph.capture_begin()
            try:
                B.nuts_set_stream(stream)
                B.nuts_sample(tgt, n_chains, n_iters, w.step_size, w.max_tree_depth, w.seed, out=out)
            finally:
                graph.capture_end()
        runs = []
        for _ in range(replays):
            for t in out:
                t.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            runs.append([t.cpu().numpy() for t in out])
            B.nuts_set_stream(None)
            between()
            torch.cuda.synchronize()
    finally:
        B.nuts_set_stream(None)
    return runs


def test_rows_stay_whole_where_the_workspace_for_two_workgroups_cannot_be_had():
    w = W.small_logreg(1000, 20, seed=3)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 512, 2, 0.02, 5
    want = gpu_run(w)
    assert want[3]["grid_blocks"] == 256                          # two workgroups for every four chains
    tgt = gpu_target(w)
    more = gpu_run(w, tgt=tgt, n_chains=1000)                     # (undivided, as there is no room for 500 workgroups)
    size = workspace_of(tgt, 1)[0]                                # no allocation from here on
    for calls in (1, 2):
        got = gpu_run(w, tgt=tgt)
        assert got[3]["grid_blocks"] == 128
        assert workspace_of(tgt, 1) == (size, 1)                  # asked for once only, and what is there stays
        for x, y in zip(got[:3], want[:3]):
            assert np.array_equal(x, y)
    workspace_of(tgt, 0)
    again = lambda: np.testing.assert_array_equal(gpu_run(w, tgt=tgt, n_chains=1000)[0], more[0])
    for got in captured_run(w, tgt, 512, 2, again):
        for x, y in zip(got, want[:3]):
            assert np.array_equal(x, y)
    fresh = gpu_target(w)                                         # a refusal where there is no workspace yet
    workspace_of(fresh, size)
    assert gpu_run(w, tgt=fresh)[3]["grid_blocks"] == 128 and workspace_of(fresh)[1] == 1


# A call that does without the larger workspace is captured; the same call outside a capture then has the target grow it.
@pytest.mark.parametrize("rows", [True, False])                   # divided rows, turns
def test_a_captured_call_keeps_the_workspace_it_was_captured_with(rows):
    if rows:
        w = W.small_logreg(1000, 20, seed=3)
        w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 512, 2, 0.02, 5
        prepare = dict(n_chains=1000)
    else:
        w = W.Workload("turns", W.GAUSS_DIAG, 500, np.dtype(np.float64), 2203, 4, 0.05, 9, seed=19, scales=10.0 ** np.linspace(-1, 1, 500))
        prepare = dict(schedule=1)
    want = gpu_run(w)
    tgt = gpu_target(w)
    gpu_run(w, tgt=tgt, **prepare)
    sizes = [workspace_of(tgt)[0]]

    def between():
        for x, y in zip(gpu_run(w, tgt=tgt)[:3], want[:3]):
            assert np.array_equal(x, y)
        sizes.append(workspace_of(tgt)[0])

    for got in captured_run(w, tgt, w.n_chains, w.n_iters, between):
        for x, y in zip(got, want[:3]):
            assert np.array_equal(x, y)
    assert sizes[0] < sizes[1] == sizes[-1]                       # (it did grow, and not while a graph was captured)
    for got in captured_run(w, tgt, w.n_chains, w.n_iters, between):  # with the larger one: divided rows and turns in a graph
        for x, y in zip(got, want[:3]):
            assert np.array_equal(x, y)
    assert counts_of(tgt)[0 if rows else 2] > 0 and sizes[-1] == sizes[1]


@pytest.mark.parametrize("silent", [2, 3])                        # the first half stops sending, the second half
@pytest.mark.parametrize("n_data,dim,dtype", [(1000, 25, np.float64), (1137, 9, np.float32), (1263, 65, np.float64)])
def test_a_workgroup_whose_partner_falls_silent_goes_on_alone(n_data, dim, dtype, silent):
    import ctypes as C
    w = W.small_logreg(n_data, dim, seed=dim, dtype=dtype)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 11, 4, 0.7 / np.sqrt(n_data), 5
    tgt, B = gpu_target(w), N()
    pairs = gpu_run(w, tgt=tgt)
    assert counts_of(tgt)[:2] == (3, 0)                           # pairs that met, and that were left
    B._check(B.lib().nuts_debug_wide_apart(tgt.handle, C.c_int(silent)))
    alone = gpu_run(w, tgt=tgt)
    assert counts_of(tgt)[:2] == (3, 3)
    for x, y in zip(alone[:3], pairs[:3]):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("n_data,dim", [(37, 33), (300, 100), (2000, 60), (5000, 40)])
def test_wide_kernel_gradients_are_as_exact_as_the_general_kernels(n_data, dim):
    """One leaf of 64 leapfrog steps from points near the posterior, against the same steps in extended precision (64-bit
    mantissa, 1e-19).  What separates a kernel's end state from those is its gradients' error: the sums of the general
    wave kernel set the bar.  AUTO's kernel measured 0.98 to 1.02 times the wave kernel's error; 1.5 leaves room for chance
    in the short sums of few rows.  (Half the column sums minus sums of sign(z) F'(|z|) in place of the residuals' sums
    measured 1.5, 3.2, 8 and 17 times.)"""
    rng = np.random.default_rng(n_data)
    X, y, wt = W.logreg_data(n_data, dim, 0.5, rng, standardize=True)
    nc, steps, eps = 24, 64, 0.15 / np.sqrt(n_data)
    init = wt + rng.standard_normal((nc, dim)) * 1.5 / np.sqrt(n_data)
    w = W.Workload("one_leaf", W.LOGREG, dim, np.dtype(np.float64), nc, 1, eps, 1, seed=41, X=X, y=y, prior_scale=1.0)
    r0 = np.array([[z for i in range((dim + 1) // 2) for z in R.normal_pair(R.draw(w.seed, i, R.TAG_MOMENTUM, 0, 0, c))][:dim]
                   for c in range(nc)])
    Xl, yl = X.astype(np.longdouble), y.astype(np.longdouble)[:, None]

    def grad(th):
        return Xl.T @ (yl - 1 / (1 + np.exp(-(Xl @ th)))) - th

    ends = []
    for v in (1, -1):
        th, r = init.T.astype(np.longdouble), r0.T.astype(np.longdouble)
        g, h = grad(th), np.longdouble(v * eps)
        for _ in range(steps):
            r = r + h / 2 * g
            th = th + h * r
            g = grad(th)
            r = r + h / 2 * g
        ends.append(th.T)
    tgt = gpu_target(w)
    err = []
    for variant in (0, N().NUTS_VARIANT_WAVE):
        s, _, n, _ = gpu_run(w, tgt=tgt, variant=variant, init=init, leaf_steps=steps)
        assert (n == steps).all()
        diff = [np.asarray(s[0] - e, dtype=np.float64) for e in ends]
        moved = (np.abs(s[0] - init) > 0).any(axis=1)
        assert moved.sum() >= nc // 2
        e2 = np.minimum(*[(d ** 2).sum(axis=1) for d in diff])[moved]
        assert e2.max() < 1e-20
        err.append(float(np.sqrt(e2.mean())))
    report("one_leaf", n=n_data, d=dim, auto=err[0], wave=err[1])
    assert err[0] <= 1.5 * err[1], f"error {err[0]:.2e} against the general kernel's {err[1]:.2e}"


@pytest.mark.parametrize("dtype,n_data,dim,n_iters,schedule,sixteen", [
    (np.float64, 10, 5, 2, 0, True), (np.float64, 499, 25, 2, 0, True), (np.float64, 500, 25, 2, 0, False), (np.float64, 500, 25, 17, 0, True),
    (np.float64, 500, 25, 17, 1, False), (np.float64, 1999, 16, 2, 0, True), (np.float64, 2000, 16, 4, 0, False), (np.float64, 2000, 16, 5, 0, True),
    (np.float64, 199, 40, 2, 0, True), (np.float64, 200, 40, 2, 0, False), (np.float32, 199, 5, 2, 0, True), (np.float32, 200, 5, 2, 0, False)])
def test_lock_step_form_between_four_and_eight_chains_per_compute_unit(dtype, n_data, dim, n_iters, schedule, sixteen):
    """Where more groups of four run than there are compute units, few rows or many iterations a launch go to sixteen."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    w = wide_workload(n_data, dim, dtype, 8 * cus)
    w.max_tree_depth = 4
    tgt = gpu_target(w)
    g = gpu_run(w, tgt=tgt, n_iters=n_iters, schedule=schedule)
    assert g[3]["grid_blocks"] == (cus // 2 if sixteen else cus)
    few = gpu_run(w, tgt=tgt, n_iters=n_iters, n_chains=4 * cus)
    assert few[3]["grid_blocks"] == cus
    for k in range(3):
        assert np.array_equal(g[k][:, :4 * cus], few[k])


def test_grid_kernels_on_four_streams_give_the_bits_of_two():
    """Long runs on many rows, all columns busy, take four streams where shorter ones take two."""
    w = W.small_logreg(120000, 64, seed=78, dtype=np.float32)
    w.n_chains, w.n_iters, w.step_size, w.max_tree_depth = 1100, 18, 0.01, 2
    tgt = gpu_target(w)
    g = gpu_run(w, tgt=tgt)
    assert_grid(g[3])
    assert g[3]["leaf_slots_useful"] == g[2].sum()
    few = gpu_run(w, tgt=tgt, n_chains=140, first_chain=960)
    sync = gpu_run(w, tgt=tgt, schedule=1, n_iters=3)
    for k in range(3):
        assert np.array_equal(g[k][:, 960:], few[k]) and np.array_equal(g[k][:3], sync[k])


@pytest.mark.parametrize("form,dim,dtype", [("wide", 40, np.float64), ("wide", 100, np.float64), ("wide", 17, np.float32), ("wide", 40, np.float32),
                                            ("band", 130, np.float64), ("band", 300, np.float32), ("band", 1025, np.float64),
                                            ("chip", 20, np.float32), ("chip", 101, np.float32), ("grid", 17, np.float32), ("grid", 71, np.float32),
                                            ("elem", 513, np.float64), ("elem", 1025, np.float32), ("elem", 2048, np.float64), ("elem", 64, np.float32)])
def test_chains_that_start_far_out_or_not_finite(form, dim, dtype):
    """Infinite, NaN and overflowing starting points: their chains stay where they are, the others do not notice."""
    rng = np.random.default_rng(dim)
    huge = 1e200 if dtype is np.float64 else 1e30
    init = rng.standard_normal((13, dim)) * (3 if form == "wide" else 1)
    init[3] = huge
    init[5, dim // 2] = -huge
    init[7] = np.inf
    init[8, 0] = -np.inf
    init[10, dim - 1] = np.nan
    if form == "wide":
        w = wide_workload(90, dim, dtype, 13)
    elif form in ("chip", "grid"):
        w = wide_workload(24000 if form == "grid" else 1700 if dim == 20 else 1003, dim, dtype, 13)
        w.n_iters, w.max_tree_depth = 4, 4
    elif form == "band":
        w = W.Workload("far_band", W.GAUSS_DENSE, dim, np.dtype(dtype), 13, 4, 0.3, 6, seed=5, precision=W.ar1_precision(dim, 0.8).astype(dtype))
    else:
        w = W.Workload("far_elem", W.GAUSS_DIAG, dim, np.dtype(dtype), 13, 4, 0.3, 6, seed=5, scales=(10.0 ** rng.uniform(-1, 1, dim)).astype(dtype))
    tgt = gpu_target(w)
    for kw in (dict(), dict(sampler=SLICE, leaf_steps=3)):
        g = gpu_run(w, tgt=tgt, init=init, **kw)
        with np.errstate(all="ignore"):
            r = ref_run(w, init=init, **kw)
        if form in ("chip", "grid"):
            (assert_chip if form == "chip" else assert_grid)(g[3])
        assert np.array_equal(np.isfinite(g[0]), np.isfinite(r[0]))
        assert np.array_equal(np.isnan(g[0]), np.isnan(r[0]))
        out = [3, 5, 7, 8, 10]
        assert np.array_equal(g[1][:, out], r[1][:, out]) and np.array_equal(g[2][:, out], r[2][:, out])
        keep = [c for c in range(13) if c not in out]
        if dtype is np.float64:
            assert_parity([x[:, keep] for x in g[:3]], [x[:, keep] for x in r], F64_TOL, label=f"{w.name} {kw}")
        else:
            f32_parity([x[:, keep] for x in g[:3]], [x[:, keep] for x in r])
        if form == "wide":                                    # sixteen chains per workgroup
            more = np.concatenate([init, rng.standard_normal((2087, dim))])
            many = gpu_run(w, tgt=tgt, init=more, n_chains=2100, n_iters=2, **kw)
            for k in range(3):
                assert np.array_equal(many[k][:, :13], g[k][:2], equal_nan=k == 0)
