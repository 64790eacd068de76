"""GPU parity at the edges of the size-selected launch forms, against the fp64 oracle."""
import time

import numpy as np
import pytest
import torch

from oracle import betty_oracle as orc
from paper_2207_02849_amd import binding
from paper_2207_02849_amd import workloads as wk
from tests.util import oracle_problem, rel_l2, time_forms

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("dims,batch,loss", [
    ((16, 16, 16), 16, "ce"),                # exactly one 16-tile everywhere
    ((17, 15, 33), 31, "ce"),                # one past, one short; output beyond the narrow-output kernels
    ((2300, 17, 3), 33, "ce"),               # K of more than one round of loads per wavefront
    ((40, 24), 65, "ce"),                    # one layer, rows of the loss Hessian wider than a 16-tile
    ((40, 9), 257, "mse"),                   # ... and inside one
    ((70, 530, 260), 100, "ce"),             # 16-, 32- and 64-tiles side by side
    ((160, 160, 48), 33, "ce"),              # the most steps straight into fragments with bf16 operands (two products of five)
    ((161, 161, 48), 33, "ce"),              # ... and one product of six
    ((96, 96, 48), 20, "ce"),                # ... in fp32 (two of six)
    ((97, 97, 48), 20, "ce"),                # ... two of seven, an odd number of steps in pairs
])
def test_small_launch_forms(dims, batch, loss, prec, tol, monkeypatch):
    monkeypatch.setenv("BETTY_TUNE", "narrow=0")
    wl = wk.tiny(kind="l2", act="gelu" if len(dims) > 2 else "none", dims=dims, batch=batch, loss=loss, prec=prec)
    prob = oracle_problem(wl)
    b = binding.from_workload(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    v = np.random.default_rng(5).standard_normal(wl.d)
    for name, got, ref in (("grad", b.betty_lower_grad(w, lam), orc.lower_grad(prob, wl.w, wl.lam)[1]),
                           ("hvp", b.betty_hvp(w, lam, dev(v)), orc.hvp(prob, wl.w, wl.lam, v)),
                           ("neumann", b.betty_hypergrad_neumann(w, lam, 2, 0.02),
                            orc.hypergrad_neumann(prob, wl.w, wl.lam, 2, 0.02))):
        assert rel_l2(host(got), ref) < tol, name
    b.close()


def partial_sums(x, V, K):
    """x V of fp32 matrices as fp32 sums: K products one after the other (each multiply-add rounded once), the partial sums in order."""
    f32 = lambda y: y.astype(np.float32).astype(np.float64)
    total = 0.0
    for k in range(0, x.shape[1], K):
        part = 0.0
        for i in range(k, min(x.shape[1], k + K)):
            part = f32(part + x[:, i, None] * V[:, i])
        total = f32(total + part)
    return total


@pytest.mark.parametrize("kernel,n,K", [
    ("tile", 100, 16), ("tile", 192, 16), ("tile", 193, 16), ("tile", 250, 16),      # 16-tiles: a partial sum a step of 16 products
    ("rop", 100, 8), ("rop", 250, 16), ("grad", 100, 8), ("grad", 250, 16),      # outputs of up to 16 columns: n / 16 rounded up to 8
])
def test_fp32_sums_of_small_launches(kernel, n, K, monkeypatch):
    """One product of a single sample, read off the gradient's first row (x_0 = 1, squared errors): no further off fp64 than
    partial sums of K products.  (Chains of twice that leave it 1.09 to 1.17 times as far; the ratio scatters by 2 %.)"""
    monkeypatch.setenv("BETTY_TUNE", "linear=0,narrow=0")
    C, N = (64, 60) if kernel == "tile" else (16, 240)
    rng = np.random.default_rng(n)
    x = np.abs(rng.standard_normal((N, n))).astype(np.float32)
    x[:, 0] = 1.0
    V = rng.standard_normal((N, n, C)).astype(np.float32)
    dims = (n, C) if kernel == "tile" else (n, n, C)
    b = binding.Betty(dims, act="none" if kernel == "tile" else "relu", loss="mse", hp="l2", prec="fp32", has_bias=False, batch_train=1, batch_val=1)
    lam = torch.full((b.d,), -80.0, device="cuda")          # no decay to speak of
    w, v = torch.zeros(b.d, device="cuda"), torch.zeros(b.d, device="cuda")
    if kernel != "tile":
        w[:n * n] = torch.eye(n, device="cuda").flatten()   # a_1 = x, exactly
    got = []
    for i in range(N):
        X, t = dev(x[i:i + 1]), torch.zeros(1, C, device="cuda")
        b.set_batches(X, X, t_tr=t, t_val=t)
        (w if kernel == "grad" else v)[-n * C:] = dev(V[i].ravel())
        g = b.betty_lower_grad(w, lam) if kernel == "grad" else b.betty_hvp(w, lam, v)
        got.append(host(g)[-n * C:][:C] / 2)
    b.close()
    x, V = x.astype(np.float64), V.astype(np.float64)
    exact = np.einsum("in,inc->ic", x, V)
    ratio = np.linalg.norm(np.array(got) - exact) / np.linalg.norm(partial_sums(x, V, K) - exact)
    print(f"{ratio:.3f}", flush=True)
    assert ratio < 1.05, ratio


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("first", [1, 2])
@pytest.mark.parametrize("dims,batch,kind,act,loss,bias", [
    ((5, 16, 16), 16, "l2", "gelu", "ce", True),              # one tile, one workgroup
    ((33, 17, 15, 1), 17, "l2", "gelu", "mse", True),         # one past, one short; a sample of its own
    ((40, 130, 129, 9), 40, "reweight", "gelu", "ce", False), # more tiles than wavefronts
    ((200, 30, 64, 300), 31, "l2", "relu", "ce", True),       # an output wider than the layers, K left over
    ((9, 20, 40, 33, 20, 12, 30, 8, 5), 50, "reweight", "relu", "ce", True),   # eight layers
    ((12, 65, 20, 4), 33, "proximal", "gelu", "ce", True),
])
def test_narrow_models_in_one_workgroup(dims, batch, kind, act, loss, bias, first, prec, tol, monkeypatch):
    """All layers of 16 samples in one workgroup, against the oracle and with the launches per layer beside it."""
    wl = wk.tiny(kind=kind, act=act, dims=dims, batch=batch, loss=loss, prec=prec, has_bias=bias, hidden=40)
    prob = oracle_problem(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    v = orc.lower_grad(prob, wl.w, wl.lam)[1]
    refs = dict(grad=v, upper=orc.upper_grad(prob, wl.w)[1], hvp=orc.hvp(prob, wl.w, wl.lam, v),
                neumann=orc.hypergrad_neumann(prob, wl.w, wl.lam, 2, 0.02))
    for form in (first, 0):
        monkeypatch.setenv("BETTY_TUNE", f"narrow={form},samples=0")
        b = binding.from_workload(wl)
        got = dict(grad=b.betty_lower_grad(w, lam), upper=b.betty_upper_grad(w), hvp=b.betty_hvp(w, lam, dev(v)),
                   neumann=b.betty_hypergrad_neumann(w, lam, 2, 0.02))
        for name, ref in refs.items():
            assert rel_l2(host(got[name]), ref) < tol, (name, form)
        if act == "gelu":
            assert rel_l2(host(b.betty_hypergrad_fd(w, lam, 1, 0.02)), orc.hypergrad_fd(prob, wl.w, wl.lam, 1, 0.02, 0.01)) < 1e-4
        b.close()


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("dims,batch,bias,one", [
    ((5, 3), 20, True, True),                # fewer parameters than a wavefront, a remainder of quads
    ((64, 64), 100, False, True),            # exactly one tile
    ((65, 63), 90, True, True),              # one row past, one column short; biases
    ((128, 128), 200, False, True),          # the most parameters: every quad of every thread
    ((127, 129), 200, True, False),          # one more: two launches a step
    ((33, 20, 9), 60, True, True),           # two layers, whose second has a row-major copy
])
def test_conjugate_gradient_of_few_parameters(dims, batch, bias, one, prec, tol, monkeypatch):
    """Step and direction in one launch: against the oracle, and the number of launches."""
    monkeypatch.setenv("BETTY_TUNE", "linear=0,narrow=0")
    wl = wk.tiny(kind="l2", act="none" if len(dims) == 2 else "gelu", dims=dims, batch=batch, prec=prec, has_bias=bias)
    wl.lam = wl.lam + 5.0                    # a definite problem
    prob = oracle_problem(wl)
    b = binding.from_workload(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    for K in (1, 2, 4):
        ref = orc.hypergrad_cg(prob, wl.w, wl.lam, K)
        for _ in range(3):                   # (the third is a replay)
            assert rel_l2(host(b.betty_hypergrad_cg(w, lam, K)), ref) < tol, K
    b.profile(True)
    b.betty_hypergrad_cg(w, lam, 4)
    assert sum(r[0] == "vector" for r in b.profile_records()) == (4 if one else 7)
    b.close()


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("first", [1, 2])
@pytest.mark.parametrize("dims,batch,kind,act,loss,bias", [
    ((5, 16, 16), 16, "l2", "gelu", "ce", True),              # one tile, one workgroup
    ((33, 17, 15, 1), 17, "l2", "gelu", "mse", True),         # one past, one short; a sample of its own
    ((40, 100, 33, 9), 40, "reweight", "gelu", "ce", False),  # more products with the direction (21) than wavefronts
    ((20, 300, 10), 40, "l2", "gelu", "ce", True),            # more tiles in a link (19, 20) than wavefronts, LDS nearly full
    ((130, 30, 64, 70), 31, "l2", "relu", "ce", True),        # an output wider than a wavefront, K left over
    ((9, 20, 40, 33, 20, 12, 30, 8, 5), 50, "reweight", "relu", "ce", True),   # eight layers
    ((12, 65, 20, 4), 33, "proximal", "gelu", "mse", True),
    ((1030, 8, 3), 20, "reweight", "gelu", "mse", True),      # many steps of K in one tile
])
def test_narrow_models_with_weights_in_lds(dims, batch, kind, act, loss, bias, first, prec, tol, monkeypatch):
    """The forward-over-reverse pass with everything in LDS before the chain begins, against the oracle; and that this is the
    form that ran: one launch where the others make one a layer."""
    wl = wk.tiny(kind=kind, act=act, dims=dims, batch=batch, loss=loss, prec=prec, has_bias=bias, hidden=40)
    prob = oracle_problem(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    v = orc.lower_grad(prob, wl.w, wl.lam)[1]
    refs = dict(hvp=orc.hvp(prob, wl.w, wl.lam, v), mixed=orc.mixed_vjp(prob, wl.w, wl.lam, v),
                neumann=orc.hypergrad_neumann(prob, wl.w, wl.lam, 2, 0.02))
    monkeypatch.setenv("BETTY_TUNE", f"narrow={first + 2},samples=0")
    b = binding.from_workload(wl)
    for _ in range(2):                                        # (a second call finds what the first left in the workspace)
        got = dict(hvp=b.betty_hvp(w, lam, dev(v)), mixed=b.betty_mixed_vjp(w, lam, dev(v)), neumann=b.betty_hypergrad_neumann(w, lam, 2, 0.02))
        for name, ref in refs.items():
            assert rel_l2(host(got[name]), ref) < tol, name
    b.profile(True)
    b.betty_hvp(w, lam, dev(v))
    kinds = [r[0] for r in b.profile_records()]
    assert kinds.count("gemm_rfwd") == (2 if first == 2 and len(dims) > 3 else 1) and "gemm_rbwd" not in kinds, kinds
    b.close()


def test_narrow_models_with_weights_in_lds_are_as_exact_as_launches(monkeypatch):
    """(as test_narrow_models_are_as_exact_as_launches)"""
    errors = {3: [], 0: []}
    for seed, dims in enumerate([(300, 24, 24, 5), (200, 40, 40, 10), (100, 17, 33, 3), (64, 64, 64, 8), (200, 30, 30, 30, 30, 4), (100, 80, 20, 40)] * 2):
        wl = wk.tiny(kind="l2", act="gelu", dims=dims, batch=100 + 31 * seed, prec="fp32", seed=seed)
        prob = oracle_problem(wl)
        v = np.random.default_rng(seed).standard_normal(wl.d).astype(np.float32)
        ref = orc.hvp(prob, wl.w, wl.lam, v.astype(np.float64))
        for form in errors:
            monkeypatch.setenv("BETTY_TUNE", f"narrow={form}")
            b = binding.from_workload(wl)
            errors[form].append(rel_l2(host(b.betty_hvp(dev(wl.w), dev(wl.lam), dev(v))), ref))
            b.close()
    ratio = np.exp(np.mean(np.log(errors[3])) - np.mean(np.log(errors[0])))
    print(f"{ratio:.3f}", flush=True)
    assert ratio < 1.05, ratio


def test_narrow_models_are_as_exact_as_launches(monkeypatch):
    """fp32 sums of all layers in one workgroup: no further off fp64 than those of the launches, on the geometric mean (one
    accumulator for a whole sum: 1.2 times as far; single results scatter by half as much)."""
    errors = {1: [], 0: []}
    for seed, dims in enumerate([(600, 24, 24, 5), (300, 40, 40, 10), (500, 17, 33, 3), (64, 64, 64, 64, 8), (200, 30, 30, 30, 30, 4), (100, 90, 20, 60)] * 2):
        wl = wk.tiny(kind="l2", act="gelu", dims=dims, batch=100 + 31 * seed, prec="fp32", seed=seed)
        prob = oracle_problem(wl)
        v = np.random.default_rng(seed).standard_normal(wl.d).astype(np.float32)
        refs = orc.lower_grad(prob, wl.w, wl.lam)[1], orc.hvp(prob, wl.w, wl.lam, v.astype(np.float64))
        for form in errors:
            monkeypatch.setenv("BETTY_TUNE", f"narrow={form}")
            b = binding.from_workload(wl)
            w, lam = dev(wl.w), dev(wl.lam)
            errors[form] += [rel_l2(host(got), ref) for got, ref in zip((b.betty_lower_grad(w, lam), b.betty_hvp(w, lam, dev(v))), refs)]
            b.close()
    ratio = np.exp(np.mean(np.log(errors[1])) - np.mean(np.log(errors[0])))
    print(f"{ratio:.3f}", flush=True)
    assert ratio < 1.05, ratio


@pytest.mark.parametrize("dims,batch,prec,act", [
    ((44, 40, 40, 40, 10), 60000, "bf16", "gelu"),
    ((117, 58, 46, 154), 29661, "bf16", "relu"),                     # one workgroup for 16 samples 1.4 times the time of the launches
    ((9, 67, 67, 41, 26, 153), 13003, "bf16", "relu"),               # ... 1.2
])
def test_narrow_models_with_many_samples_go_by_launches(dims, batch, prec, act, monkeypatch):
    """Beyond a workgroup per compute unit the launches per layer fill the chip, and the rule knows the batch."""
    rule, launches = time_forms(monkeypatch, lambda b, w: b.betty_hypergrad_neumann(w, w, 9, 1e-4), ("samples=0", "narrow=0,samples=0"), rounds=5,
                                reps=3, dims=dims, act=act, loss="ce", hp="l2", prec=prec, batch_train=batch, batch_val=batch)
    assert rule < 1.1 * launches, (rule, launches)        # (first-order passes may be a few percent slower, runs differ by as much)


@pytest.mark.parametrize("dims,batch,K", [((1006, 9, 80), 65, 9), ((915, 33, 33, 146), 25, 9)])     # 1.25 times the time of the series over samples
def test_narrow_models_keep_the_series_over_samples_where_it_is_faster(dims, batch, K, monkeypatch):
    rule, samples = time_forms(monkeypatch, lambda b, w: b.betty_hypergrad_neumann(w, w[:b.n_hyper], K, 1e-4), ("", "narrow=0"), dims=dims,
                               act="gelu", loss="ce", hp="reweight", prec="fp32" if len(dims) == 3 else "bf16", batch_train=batch, batch_val=batch)
    assert rule < 1.1 * samples, (rule, samples)


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("dims,batch,kind,samples", [
    ((12, 257, 3), 521, "reweight", 0),      # one column in the second block
    ((20, 300, 7), 530, "l2", 0),
    ((12, 512, 16), 521, "reweight", 1),     # both blocks whole; the series over samples
])
def test_narrow_outputs_with_a_second_block_of_columns(dims, batch, kind, samples, prec, tol, monkeypatch):
    """With more than 512 samples a workgroup takes all columns of a hidden layer beyond 256, a wavefront two blocks of 16."""
    monkeypatch.setenv("BETTY_TUNE", f"narrow=0,samples={samples}")
    wl = wk.tiny(kind=kind, act="gelu", dims=dims, batch=batch, prec=prec, hidden=40)
    prob = oracle_problem(wl)
    b = binding.from_workload(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    v = np.random.default_rng(3).standard_normal(wl.d)
    for name, got, ref in (("grad", b.betty_lower_grad(w, lam), orc.lower_grad(prob, wl.w, wl.lam)[1]),
                           ("hvp", b.betty_hvp(w, lam, dev(v)), orc.hvp(prob, wl.w, wl.lam, v)),
                           ("neumann", b.betty_hypergrad_neumann(w, lam, 2, 0.02), orc.hypergrad_neumann(prob, wl.w, wl.lam, 2, 0.02))):
        assert rel_l2(host(got), ref) < tol, name
    b.profile(True)
    b.betty_hypergrad_neumann(w, lam, 2, 0.02)
    assert [r[0] for r in b.profile_records()].count("last_layer") >= 3        # gradient, two products
    b.close()


@pytest.mark.parametrize("dims,batch,batch_val,K", [                                     # on parameters:
    ((232, 56, 46), 124, 350, 9), ((413, 14, 38), 331, 78, 20), ((511, 12, 34), 50, 60, 9),      # 1.20, 1.13, 1.4 times the time
])
def test_series_over_samples_beside_passes_with_weights_in_lds(dims, batch, batch_val, K, monkeypatch):
    rule, samples = time_forms(monkeypatch, lambda b, w: b.betty_hypergrad_neumann(w, w[:b.n_hyper], K, 1e-4), ("", "samples=1"), dims=dims,
                               act="relu", loss="ce", hp="reweight", prec="fp32", batch_train=batch, batch_val=batch_val)
    assert rule < 1.08 * samples, (rule, samples)          # (the same form: 1.0)


@pytest.mark.parametrize("kind", ["l2", "reweight"])
@pytest.mark.parametrize("batch,batch_val", [(13000, 50), (40, 24600), (40, 50)])
def test_finite_differences_of_narrow_models_mix_forms(batch, batch_val, kind, monkeypatch):
    """The pass at w, those at both points and the shared first layer with either form of pass beside the other."""
    monkeypatch.setenv("BETTY_TUNE", "layer1=1")
    wl, big = (wk.tiny(kind=kind, act="gelu", dims=(20, 12, 16, 12, 20), batch=n, hidden=20, seed=s) for n, s in ((batch, 0), (batch_val, 3)))
    wl.X_val, wl.y_val = big.X_val, big.y_val
    prob = oracle_problem(wl)
    b = binding.from_workload(wl)
    for K in (0, 1, 2):                                    # (tolerances as in test_finite_difference_forms)
        assert rel_l2(host(b.betty_hypergrad_fd(dev(wl.w), dev(wl.lam), K, 0.05, 0.01)),
                      orc.hypergrad_fd(prob, wl.w, wl.lam, K, 0.05, 0.01)) < (1e-3 if kind == "reweight" else 1e-4), K
    b.close()


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("kind,samples", [("l2", 0), ("reweight", 1)])
@pytest.mark.parametrize("dims,batch", [
    ((64, 64, 64, 40), 64),                  # whole tiles, one k-tile a group
    ((65, 33, 130, 17), 63),                 # ragged rows, columns and K
    ((1100, 300, 31), 129),                  # the long-loop form in some products, not in others; Hessian in the epilogue
])
def test_two_way_split_of_64_tiles(dims, batch, kind, samples, prec, tol, monkeypatch):
    """Against the oracle, and other bits than those of unsplit 64-tiles: the sums along K are grouped by halves (a bf16
    series whose sums fit one k-tile has the same)."""
    wl = wk.tiny(kind=kind, act="gelu", dims=dims, batch=batch, prec=prec)
    prob = oracle_problem(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    v = orc.lower_grad(prob, wl.w, wl.lam)[1]
    refs = dict(grad=v, hvp=orc.hvp(prob, wl.w, wl.lam, v), neumann=orc.hypergrad_neumann(prob, wl.w, wl.lam, 2, 0.02))
    got = {}
    for form in ("pair=1", "blocks=1"):
        monkeypatch.setenv("BETTY_TUNE", f"{form},narrow=0,samples={samples}")
        b = binding.from_workload(wl)
        got[form] = dict(grad=host(b.betty_lower_grad(w, lam)), hvp=host(b.betty_hvp(w, lam, dev(v))),
                         neumann=host(b.betty_hypergrad_neumann(w, lam, 2, 0.02)))
        for name, ref in refs.items():
            assert rel_l2(got[form][name], ref) < tol, (name, form)
        b.close()
    for name in ("grad", "hvp"):
        assert not np.array_equal(got["pair=1"][name], got["blocks=1"][name]), name


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("loss", ["ce", "mse"])
@pytest.mark.parametrize("C,batch", [(64, 5), (65, 16), (256, 15), (257, 33), (1024, 17), (1100, 18)])
def test_loss_rows_of_wide_outputs(C, batch, loss, prec, tol, monkeypatch):
    """Outputs at the edges of what a wavefront keeps of a row and of a workgroup's columns and samples."""
    monkeypatch.setenv("BETTY_TUNE", "narrow=0")
    wl = wk.tiny(kind="l2", act="gelu", dims=(9, 20, C), batch=batch, loss=loss, prec=prec)
    prob = oracle_problem(wl)
    b = binding.from_workload(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    v = np.random.default_rng(C).standard_normal(wl.d)
    loss_ref, grad_ref = orc.lower_grad(prob, wl.w, wl.lam)
    grad, cost = b.betty_lower_grad(w, lam, want_loss=True)
    assert rel_l2(host(grad), grad_ref) < tol and abs(float(cost) - loss_ref) < tol * abs(loss_ref)
    b.profile(True)
    assert rel_l2(host(b.betty_hvp(w, lam, dev(v))), orc.hvp(prob, wl.w, wl.lam, v)) < tol
    assert sum(r[0] == "loss" for r in b.profile_records()) == 2       # the rows of the loss and those of its Hessian
    b.close()


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("layers", [2, 4, 5, 8, 9])
def test_operand_conversions_at_the_edges_of_a_launch(layers, prec, tol):
    """Four matrices are the most of the short form of a conversion, sixteen those of a launch: a gradient converts one a
    layer, a product two."""
    wl = wk.tiny(kind="l2", act="gelu", dims=(21, 18) + (14, 17) * (layers // 2 - 1) + (13,) * (layers % 2) + (5,), batch=20, prec=prec)
    assert len(wl.dims) == layers + 1
    prob = oracle_problem(wl)
    b = binding.from_workload(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    v = orc.lower_grad(prob, wl.w, wl.lam)[1]
    for matrices, call, ref in ((layers, lambda: b.betty_lower_grad(w, lam), v),
                                (2 * layers, lambda: b.betty_hvp(w, lam, dev(v)), orc.hvp(prob, wl.w, wl.lam, v))):
        b.profile(True)
        assert rel_l2(host(call()), ref) < tol
        assert sum(r[0] == "shadow" for r in b.profile_records()) == -(-matrices // 16)
        b.profile(False)
    b.close()


def test_recorded_calls_follow_streams_and_batches():
    """A handle without an explicit stream runs on the caller's current stream; recorded sequences
    survive a move to another stream and new batches (labels included), and one argument set does
    not push out another."""
    wl, wl2 = (wk.tiny(kind="reweight", dims=(40, 30, 5), batch=33, hidden=9, seed=s) for s in (0, 1))
    batches = [dict(X_tr=dev(x.X_tr), X_val=dev(x.X_val), y_tr=torch.as_tensor(x.y_tr).int().cuda(),
                    y_val=torch.as_tensor(x.y_val).int().cuda()) for x in (wl, wl2)]
    b = binding.from_workload(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    outs = [torch.empty(b.n_hyper, device="cuda") for _ in range(2)]
    other = torch.cuda.Stream()
    ref = [orc.hypergrad_neumann(oracle_problem(x), wl.w, wl.lam, 3, 0.05) for x in (wl, wl2)]
    for rep in range(4):
        for batch, want in zip(batches, ref):
            b.set_batches(**batch)
            for out in outs:
                if rep % 2:
                    other.wait_stream(torch.cuda.current_stream())
                    with torch.cuda.stream(other):
                        b.betty_hypergrad_neumann(w, lam, 3, 0.05, out=out)
                    torch.cuda.current_stream().wait_stream(other)
                else:
                    b.betty_hypergrad_neumann(w, lam, 3, 0.05, out=out)
                assert rel_l2(host(out), want) < 1e-4
                out.zero_()
    out = b.betty_hypergrad_neumann(w, lam, 3, 0.05)
    b.stream.synchronize()                       # the handle's own stream is ordered behind the call
    assert rel_l2(out.cpu().numpy(), ref[1]) < 1e-4
    b.close()


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("kind", ["reweight", "proximal"])
def test_series_with_many_validation_samples(kind, prec, tol, monkeypatch):
    """Far more validation than train samples: both forms of the series agree with the oracle, and the
    rule counts what they cost at the beginning of a call (one step: parameter-sized; a dense vector
    in place of the validation gradient does not see them)."""
    wl = wk.tiny(kind=kind, act="gelu", dims=(256, 128, 128, 10), batch=64, prec=prec, hidden=20, prox_rho=0.3)
    big = wk.tiny(kind=kind, act="gelu", dims=(256, 128, 128, 10), batch=16384, prec=prec, hidden=20, seed=3)
    wl.X_val, wl.y_val = big.X_val, big.y_val
    prob = oracle_problem(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    u = dev(np.random.default_rng(2).standard_normal(wl.d))
    got = {}
    for form in ("samples=0", "samples=1", ""):
        monkeypatch.setenv("BETTY_TUNE", form)
        b = binding.from_workload(wl)
        got[form] = [host(b.betty_hypergrad_neumann(w, lam, K, 0.02)) for K in (1, 3)] + \
                    [host(b.betty_best_response_neumann(w, lam, u, 10, 0.02))]
        b.close()
    for k, K in enumerate((1, 3)):
        ref = orc.hypergrad_neumann(prob, wl.w, wl.lam, K, 0.02)
        for form in got:
            assert rel_l2(got[form][k], ref) < tol, (form, K)
    assert np.array_equal(got[""][0], got["samples=0"][0]) and not np.array_equal(got[""][0], got["samples=1"][0])
    if kind == "reweight" and prec == "fp32":
        assert np.array_equal(got[""][2], got["samples=1"][2]) and not np.array_equal(got[""][2], got["samples=0"][2])


def test_proximal_series_factors_are_rounded_once(monkeypatch):
    """The factors in front of the proximal result, 2 rho alpha sum_j beta^j and 2 rho alpha^2, are formed in double
    and rounded once: an error in them is one of the whole result (1.3e-7 for these numbers in 32-bit
    steps), unlike the roundings of its elements, which average out of the projection on the oracle's.
    (The oracle takes rho and alpha as the 32-bit numbers that the library is given; 128 validation
    samples, so that the mean over them rounds nothing.)"""
    rho, alpha = float(np.float32(0.1)), float(np.float32(0.1))
    wl = wk.tiny(kind="proximal", act="gelu", dims=(300, 200, 10), batch=126, prec="fp32", prox_rho=rho)
    prob = oracle_problem(wl)
    ref = orc.hypergrad_neumann(prob, wl.w, wl.lam, 5, alpha)
    monkeypatch.setenv("BETTY_TUNE", "samples=1")
    b = binding.from_workload(wl)
    got = host(b.betty_hypergrad_neumann(dev(wl.w), dev(wl.lam), 5, alpha))
    err = abs(np.vdot(got, ref) / np.vdot(ref, ref) - 1.0)            # the error common to all elements
    print(f"{err:.2e}", flush=True)
    assert err < 8e-8                   # 6e-8 of the first factor, as much of the second one's third of the result
    b.close()


def test_stream_of_a_handle_kept_from_before_a_call():
    """A reference to `stream` taken earlier is as good as a fresh one: waiting for it, or queueing work
    on it, covers the calls made since."""
    wl = wk.tiny(kind="l2", act="gelu", dims=(2048, 2048, 10), batch=256, prec="fp32")
    b = binding.from_workload(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    kept = b.stream
    out = torch.empty(b.n_hyper, device="cuda")
    b.betty_hypergrad_neumann(w, lam, 20, 0.01, out=out)
    want = out.clone()
    torch.cuda.synchronize()
    for use in ("synchronize", "record_event", "wait_stream", "stream"):
        for _ in range(3):                        # several milliseconds of work
            b.betty_hypergrad_neumann(w, lam, 20, 0.01, out=out)
        behind = torch.cuda.current_stream().record_event()
        if use == "synchronize":
            kept.synchronize()
        elif use == "record_event":
            kept.record_event().synchronize()
        elif use == "wait_stream":
            other = torch.cuda.Stream()
            other.wait_stream(kept)
            other.synchronize()
        else:
            with torch.cuda.stream(kept):
                copy = out.clone()
            kept.synchronize()
            assert torch.equal(copy, want)
        assert behind.query(), use
    b.close()
    kept.synchronize()                            # the stream outlives the handle


DEEP = (24, 20, 20, 20, 20, 20, 20, 4)               # ten launches a call and more, layer by layer: recorded when they repeat


def launches(b, call):
    b.profile(True)
    call()
    n = len(b.profile_records())
    b.profile(False)
    return n


@pytest.mark.parametrize("dims,act,repeats", [((64, 32, 4), "relu", 2), (DEEP, "gelu", 2), (DEEP, "gelu", 3)])
def test_steps_whose_arguments_keep_changing(dims, act, repeats, monkeypatch):
    """Two or three steps with each learning rate cost what steps with as many learning rates cost (next to
    nothing is recorded that will not be replayed), and each uses the scalars it was given."""
    monkeypatch.setenv("BETTY_TUNE", "narrow=0")
    wl = wk.tiny(kind="l2", act=act, dims=dims, batch=64, prec="fp32")
    prob = oracle_problem(wl)
    b = binding.from_workload(wl)
    w, lam, mom = dev(wl.w), dev(wl.lam), torch.zeros(wl.d, device="cuda")
    n = launches(b, lambda: b.betty_lower_sgd_step(w.clone(), lam, mom.clone(), 0.0, 0.0))
    assert n >= 10 if dims == DEEP else n < 10, n
    w64, m64 = wl.w.astype(np.float64), np.zeros(wl.d)
    for k in range(8):
        lr, wd = 0.02 / (1 + k // repeats), 0.01 * (k // repeats)
        b.betty_lower_sgd_step(w, lam, mom, lr, 0.9, wd)
        w64, m64 = orc.lower_sgd_step(prob, w64, wl.lam.astype(np.float64), m64, lr, 0.9, wd)
        assert rel_l2(host(w), w64) < 1e-5 and rel_l2(host(mom), m64) < 1e-4, k
    rates = iter(1e-6 * np.arange(1, 10000))

    def loop(steps_per_rate):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(120 // steps_per_rate):
            lr = float(next(rates))
            for _ in range(steps_per_rate):
                b.betty_lower_sgd_step(w, lam, mom, lr, 0.0)
        torch.cuda.synchronize()
        return time.perf_counter() - t0

    # The card alternates, for seconds at a time, between two speeds of short launches (steps of 64-32-4 14.8 and 18.5 us, 1.25 times, whatever the
    # loop), so loops are compared with those beside them and not the fastest of either.
    both = [(loop(1), loop(repeats)) for _ in range(30)]
    ratio = float(np.median([many / one for one, many in both]))
    assert ratio < 1.25, (ratio, both)            # (recording every second step: 1.6 times)
    b.close()


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
def test_short_calls_that_are_recorded(prec, tol, monkeypatch):
    """Gradients, products and steps of a deep small model are replayed from the third call on: every call
    against the oracle, with other batches registered and another stream in between."""
    monkeypatch.setenv("BETTY_TUNE", "narrow=0")
    wl, wl2 = (wk.tiny(kind="reweight", act="gelu", dims=DEEP, batch=33, prec=prec, hidden=9, seed=s) for s in (0, 1))
    wl2.w, wl2.lam = wl.w, wl.lam
    batches = [dict(X_tr=dev(x.X_tr), X_val=dev(x.X_val), y_tr=torch.as_tensor(x.y_tr).int().cuda(),
                    y_val=torch.as_tensor(x.y_val).int().cuda()) for x in (wl, wl2)]
    probs = [oracle_problem(x) for x in (wl, wl2)]
    b = binding.from_workload(wl)
    w, lam, w2, mom = dev(wl.w), dev(wl.lam), dev(wl.w), torch.zeros(wl.d, device="cuda")
    v = np.random.default_rng(5).standard_normal(wl.d).astype(np.float32)
    q = orc.upper_grad(probs[0], wl.w)[1].astype(np.float32)
    vd, qd, Hv, m = dev(v), dev(q), torch.empty_like(w), torch.empty_like(lam)
    grad, gval = torch.empty_like(w), torch.empty_like(w)
    other, lib = torch.cuda.Stream(), b.lib
    for call in (lambda: b.betty_hvp(w, lam, vd, out=Hv), lambda: b.betty_lower_grad(w, lam), lambda: b.betty_upper_grad(w),
                 lambda: b.betty_mixed_vjp(w, lam, qd), lambda: b.betty_lower_sgd_step(w2.clone(), lam, mom.clone(), 0.0, 0.0)):
        assert launches(b, call) >= 10
    w64, m64 = wl.w.astype(np.float64), np.zeros(wl.d)
    for rep in range(7):
        prob = probs[rep % 2]
        b.set_batches(**batches[rep % 2])
        for t in (Hv, m, grad, gval):
            t.zero_()
        use = other if rep in (3, 5) else torch.cuda.current_stream()
        use.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(use):
            b.betty_hvp(w, lam, vd, out=Hv)
            b._call(lib.betty_lower_grad, w.data_ptr(), lam.data_ptr(), grad.data_ptr(), None)
            b._call(lib.betty_upper_grad, w.data_ptr(), gval.data_ptr(), None)
            b._call(lib.betty_mixed_vjp, w.data_ptr(), lam.data_ptr(), qd.data_ptr(), m.data_ptr())
            b.betty_lower_sgd_step(w2, lam, mom, 0.05, 0.9, 1e-3)
        torch.cuda.current_stream().wait_stream(use)
        w64, m64 = orc.lower_sgd_step(prob, w64, wl.lam.astype(np.float64), m64, 0.05, 0.9, 1e-3)
        for name, got, ref in (("hvp", Hv, orc.hvp(prob, wl.w, wl.lam, v)), ("lower", grad, orc.lower_grad(prob, wl.w, wl.lam)[1]),
                               ("upper", gval, orc.upper_grad(prob, wl.w)[1]), ("mixed", m, orc.mixed_vjp(prob, wl.w, wl.lam, q)),
                               ("w", w2, w64), ("momentum", mom, m64)):
            assert rel_l2(host(got), ref) < tol, (rep, name)
    b.close()


def test_chain_leaves_the_finetune_handle_on_its_stream():
    """Only the pretrain handle is moved to another stream: the finetune handle's calls after the chain
    run where they ran before, not behind what the pretrain handle does next."""
    pre_wl, ft_wl = wk.chain3(seed=3, act="gelu", skip_last=True)
    home, other = torch.cuda.Stream(), torch.cuda.Stream()
    pre, ft = binding.from_workload(pre_wl, stream=home), binding.from_workload(ft_wl, stream=home)
    lib = pre.lib
    w, theta, v = dev(pre_wl.w), dev(pre_wl.lam), dev(ft_wl.w)
    want = ft.betty_lower_grad(v, w)
    got, dtheta = torch.zeros_like(want), torch.zeros(pre.n_hyper, device="cuda")
    busy = torch.zeros(64 << 20, device="cuda")
    torch.cuda.synchronize()
    chain = lambda: pre._check(lib.betty_hypergrad_chain3(pre.h, ft.h, w.data_ptr(), theta.data_ptr(), v.data_ptr(),
                                                          2, 0.05, 2, 0.05, dtheta.data_ptr()))
    pre._check(lib.betty_run_on(pre.h, other.cuda_stream))
    chain()
    ref = host(dtheta)
    for _ in range(3):
        got.zero_(), dtheta.zero_()
        torch.cuda.synchronize()
        chain()
        with torch.cuda.stream(other):
            for _ in range(100):
                busy.add_(1.0)                    # about ten milliseconds
        ft._check(lib.betty_lower_grad(ft.h, v.data_ptr(), w.data_ptr(), got.data_ptr(), None))
        home.synchronize()
        assert torch.equal(got, want)             # (not yet there if the gradient were queued on `other`)
        assert rel_l2(host(dtheta), ref) < 1e-6
    torch.cuda.synchronize()
    pre.close()
    ft.close()


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("kind,dims,batch,act", [
    ("reweight", (40, 33), 65, "none"),                          # one layer: no link at all
    ("reweight", (40, 9), 20, "none"),                           # ... with a narrow output
    ("reweight", (300, 200, 150, 10), 130, "relu"),              # narrow output; batch of two padded 64-groups and a bit
    ("reweight", (70, 200, 90, 20), 64, "gelu"),                 # wide output
    ("proximal", (30, 31, 32, 33, 34, 35, 36, 37, 38, 5), 40, "gelu"),   # more layers than a launch has problems
    ("proximal", (300, 150, 10), 129, "gelu"),
    ("proximal", (33, 130, 40), 7, "none"),
])
def test_series_in_sample_space(kind, dims, batch, act, prec, tol, monkeypatch):
    """Costs without a per-parameter diagonal carry the Neumann series over pairs of samples; forced on here,
    from the validation gradient and from a dense vector, against the oracle and (where a family of
    inputs is outside the tolerance in either form) no worse than the parameter-sized form."""
    wl = wk.tiny(kind=kind, act=act, dims=dims, batch=batch, prec=prec, hidden=20, prox_skip_last=len(dims) > 3, prox_rho=0.3)
    prob = oracle_problem(wl)
    u = orc.lower_grad(prob, wl.w, wl.lam)[1].astype(np.float32)
    err = {}
    for form in (0, 1, 2):
        # (2: first-order passes with all layers in one workgroup, where the model has up to eight)
        monkeypatch.setenv("BETTY_TUNE", f"samples={min(form, 1)},narrow={form // 2}")
        b = binding.from_workload(wl)
        w, lam = dev(wl.w), dev(wl.lam)
        for K in (0, 1, 4):
            err[form, K] = max(
                rel_l2(host(b.betty_hypergrad_neumann(w, lam, K, 0.05)), orc.hypergrad_neumann(prob, wl.w, wl.lam, K, 0.05)),
                rel_l2(host(b.betty_best_response_neumann(w, lam, dev(u), K, 0.05)),
                       orc.best_response_neumann(prob, wl.w, wl.lam, u.astype(np.float64), K, 0.05)))
        b.close()
    for K in (0, 1, 4):
        assert max(err[1, K], err[2, K]) < max(tol, 1.5 * err[0, K]), (K, err)


@pytest.mark.parametrize("kind,dims,batch", [
    ("l2", (65, 3), 40),                     # widths that allow no 16-byte accesses, a second tile of one row
    ("l2", (64, 64), 100),                   # exactly one tile
    ("l2", (130, 68), 300),
    ("proximal", (70, 67), 90),
    ("reweight", (33, 10), 65),
])
def test_conjugate_gradient_steps(kind, dims, batch):
    """K = 0 (no step), 1 (the first is the last), 2 and 4 steps of the fused vector updates."""
    wl = wk.tiny(kind=kind, act="none", dims=dims, batch=batch, hidden=20, prox_rho=0.3)
    prob = oracle_problem(wl)
    b = binding.from_workload(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    for K in (0, 1, 2, 4):
        got, ref = host(b.betty_hypergrad_cg(w, lam, K)), orc.hypergrad_cg(prob, wl.w, wl.lam, K)
        assert np.abs(got).max() == 0 if K == 0 else rel_l2(got, ref) < 1e-4, K
    b.close()


@pytest.mark.parametrize("layer1", (0, 1))
@pytest.mark.parametrize("paired", (0, 1))
@pytest.mark.parametrize("kind,dims,batch", [
    ("l2", (65, 3), 40),                     # one layer; rows that allow no 16-byte accesses, a second tile of one row
    ("l2", (64, 64, 20), 64),                # exactly one tile
    ("l2", (70, 130, 68, 9), 129),           # ragged tiles, batch one past two 64-groups
    ("proximal", (33, 66, 10), 31),
    ("reweight", (33, 66, 10), 65),
])
def test_finite_difference_forms(kind, dims, batch, paired, layer1, monkeypatch):
    """Both points of a central difference in shared launches, and one after the other; layer 1 of both from one product
    or from their own weights."""
    wl = wk.tiny(kind=kind, act="gelu" if len(dims) > 2 else "none", dims=dims, batch=batch, hidden=20, prox_rho=0.3)
    prob = oracle_problem(wl)
    monkeypatch.setenv("BETTY_TUNE", f"fd2={paired},layer1={layer1},narrow=0")
    b = binding.from_workload(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    for K in (0, 1, 3):
        # the fp32 gradients' rounding (2^-24) over 2 eps |v| = 0.02, times alpha: some 1e-6; reweighting ends in a
        # difference of losses of order 1 by 0.02 <grad l, q/|q|>: 2^-23 / 0.02 over a projection of some 0.1, 1e-4
        assert rel_l2(host(b.betty_hypergrad_fd(w, lam, K, 0.05, 0.01)),
                      orc.hypergrad_fd(prob, wl.w, wl.lam, K, 0.05, 0.01)) < (1e-3 if kind == "reweight" else 1e-4), K
    b.close()


def test_sums_beside_the_weight_gradients_keep_small_terms():
    """The regulariser's cost is summed inside the weight-gradient launch: a lane adds at most the 64 terms of one
    tile in fp32, tiles and lanes are added in double.  67M weights of size 1, on 4096 tiles of 128 that 512
    workgroups walk, eight each; in its first tile every lane meets one weight of 4096, whose square is 2^24, beside
    which a square of 1 is lost in fp32: 63 of 2^24 where the sum stays within a tile (3.8e-6), 511 where it does
    not (3e-5).  Zero inputs leave the data term at log(16384)."""
    n_in, n_out, B = 4096, 16384, 4
    b = binding.Betty((n_in, n_out), act="none", loss="ce", hp="l2", prec="bf16", has_bias=False, batch_train=B, batch_val=B)
    r, c = torch.arange(n_in, device="cuda")[:, None], torch.arange(n_out, device="cuda")[None, :]
    big = (r < 512) & (r % 128 < 32) & (r % 4 == 0) & (c % 4 == 0)
    w = torch.where(big, 4096.0, 1.0).float().flatten()
    X, y = torch.zeros(B, n_in, device="cuda"), torch.zeros(B, dtype=torch.int32, device="cuda")
    b.set_batches(X, X, y, y)
    lam = torch.zeros_like(w)
    want = float((w.double() ** 2).sum()) + np.log(n_out)
    _, loss = b.betty_lower_grad(w, lam, want_loss=True)
    assert abs(float(loss) - want) < 1e-5 * want
    b.close()


@pytest.mark.parametrize("dims,batch", [((40, 30, 7), 33), ((300, 500, 10), 40), ((1500, 1024, 64), 32)])   # 16-, 32- and 64-tiles
def test_finite_difference_mixed_term_is_rounded_once(dims, batch):
    """The mixed term for L2 decay, -2 exp(lambda) w q, leaves in fp32 but is formed in double: half a unit in the
    last place, 2^-24, against the same product in fp64.  K = 0: q = alpha g with g the upper gradient.  K = 1: zero
    inputs make the data gradient of the first layer zero at both points, so with a step of 2^-60 its
    p = g + (g - alpha H g) is 2 g exactly."""
    wl = wk.tiny(kind="l2", act="gelu", dims=dims, batch=batch)
    b = binding.from_workload(wl)
    w, lam = dev(wl.w), dev(wl.lam)
    for K, alpha in ((0, 0.05), (1, 2.0 ** -60)):
        if K:
            y = [torch.as_tensor(a).int().cuda() for a in (wl.y_tr, wl.y_val)]
            b.set_batches(torch.zeros(batch, dims[0], device="cuda"), dev(wl.X_val), *y)
        g, got = host(b.betty_upper_grad(w)), host(b.betty_hypergrad_fd(w, lam, K, alpha, 0.01))
        n = dims[0] * dims[1]
        want = -2.0 * np.exp(wl.lam.astype(np.float64)) * wl.w.astype(np.float64) * np.float64(np.float32(alpha)) * (1 + K) * g
        big = np.abs(want[:n]) > 1e-36           # (above the range where a unit is no longer relative)
        assert big.mean() > 0.9
        assert np.abs(got[:n][big] / want[:n][big] - 1.0).max() < 1.001 * 2.0 ** -24, K
    b.close()


@pytest.mark.parametrize("n,m,tune", [
    (100, 70, ""),                           # 16-tiles; the second group of 64 samples is not full
    (64, 20, ""),                            # exactly one group
    (300, 290, ""),                          # 32-tiles
    (300, 290, ",blocks=1"),                 # 64-tiles
    (300, 290, ",wgrad128=1"),               # the 128-tile kernel, two k-tiles of padding
])
def test_proximal_series_keeps_its_sums_beyond_bf16(n, m, tune, monkeypatch):
    """In sample space the proximal cost needs sums of R a and R delta over the steps.  With unit inputs, zero weights
    and delta = c I the Hessian only swaps the two layers' directions: (H V)_1 = c V_2^T, (H V)_2 = c V_1^T.  From
    u_1 = u_2^T (powers of two) with alpha c = 1/2 every step's V is exact in bf16, u (1, 1.5, ..., 1.96875), and
    the sum of six, 10.03125 u, is not: rounded to bf16 it puts the result off by 8e-3.  Value and remainder carry
    it exactly; what is left are fp32 roundings (and the step beta = 1 - 2^-19)."""
    K, c, alpha, rho = 6, 2.0 ** -4, 8.0, 2.0 ** -23
    rng = np.random.default_rng(3)
    u1 = np.ldexp(rng.choice((-1.0, 1.0), (n, m)), rng.integers(-1, 2, (n, m)))
    u = np.concatenate([u1.ravel(), u1.T.ravel()]).astype(np.float32)
    B, X, t = n, np.eye(n), -0.5 * n * c * np.eye(n)
    monkeypatch.setenv("BETTY_TUNE", "samples=1" + tune)
    b = binding.Betty((n, m, n), act="none", loss="mse", hp="proximal", prec="bf16", has_bias=False, batch_train=B,
                      batch_val=B, prox_rho=rho)
    b.set_batches(dev(X), dev(X), t_tr=dev(t), t_val=dev(t))
    w = torch.zeros(b.d, device="cuda")
    prob = orc.Problem(dims=(n, m, n), act="none", loss="mse", hp="proximal", has_bias=False, X_tr=X, X_val=X,
                       t_tr=t, t_val=t, prox_rho=rho)
    got = host(b.betty_best_response_neumann(w, w, dev(u), K, alpha))
    ref = orc.best_response_neumann(prob, np.zeros(b.d), np.zeros(b.d), u.astype(np.float64), K, alpha)
    assert np.abs(got - ref).max() < 2e-5 * np.abs(ref).max() and rel_l2(got, ref) < 2e-5
    b.close()


@pytest.mark.parametrize("B", (32, 128))
def test_proximal_series_keeps_its_bias_sums_beyond_bf16(B, monkeypatch):
    """The same for a bias: zero inputs, squared error, H c = 2 c; with alpha = 1/4 the same six steps."""
    n_in, n_out, K, alpha, rho = 5, 40, 6, 0.25, 2.0 ** -18
    u = np.zeros(n_in * n_out + n_out, np.float32)
    u[n_in * n_out:] = np.ldexp(1.0, np.arange(n_out) % 3 - 1)
    X, t = np.zeros((B, n_in)), np.zeros((B, n_out))
    monkeypatch.setenv("BETTY_TUNE", "samples=1")
    b = binding.Betty((n_in, n_out), act="none", loss="mse", hp="proximal", prec="bf16", batch_train=B, batch_val=B,
                      prox_rho=rho)
    b.set_batches(dev(X), dev(X), t_tr=dev(t), t_val=dev(t))
    w = torch.zeros(b.d, device="cuda")
    prob = orc.Problem(dims=(n_in, n_out), act="none", loss="mse", hp="proximal", has_bias=True, X_tr=X, X_val=X,
                       t_tr=t, t_val=t, prox_rho=rho)
    got = host(b.betty_best_response_neumann(w, w, dev(u), K, alpha))
    ref = orc.best_response_neumann(prob, np.zeros(b.d), np.zeros(b.d), u.astype(np.float64), K, alpha)
    assert rel_l2(got, ref) < 2e-5
    b.close()


@pytest.mark.parametrize("dims,batch,batch_val,kind,K", [
    ((15, 1200, 86), 976, 40, "l2", 1),               # layer 1 of both points from one product: 1.2 times the time of its own
    ((168, 812, 26), 23949, 144, "reweight", 1),      # ... 1.25
    ((1011, 97, 3), 788, 203, "l2", 1),               # ... 1.16
])
def test_finite_differences_share_the_first_layer_only_where_it_is_faster(dims, batch, batch_val, kind, K, monkeypatch):
    rule, own = time_forms(monkeypatch, lambda b, w: b.betty_hypergrad_fd(w, w[:b.n_hyper], K, 1e-4), ("narrow=0", "narrow=0,layer1=0"), reps=10, dims=dims,
                           act="gelu", loss="ce", hp=kind, prec="fp32", batch_train=batch, batch_val=batch_val)
    assert rule < 1.08 * own, (rule, own)


@pytest.mark.parametrize("rows,tune", [(1000, "tile128=1"), (40, "pair=1"), (129, "blocks=1"), (129, "")])
def test_first_layer_at_both_points_in_every_tile(rows, tune, monkeypatch):
    """Large launches take 64-tiles there, also where a plain forward product takes 128-tiles; z_1 at w with a kernel of its
    own size beside a validation batch of another."""
    wl, big = (wk.tiny(kind="l2", act="gelu", dims=(140, 150, 20), batch=n, hidden=20, seed=s) for n, s in ((rows, 0), (9, 3)))
    wl.X_val, wl.y_val = big.X_val, big.y_val
    prob = oracle_problem(wl)
    monkeypatch.setenv("BETTY_TUNE", f"layer1=1,narrow=0,{tune}")
    b = binding.from_workload(wl)
    for K in (1, 2):
        assert rel_l2(host(b.betty_hypergrad_fd(dev(wl.w), dev(wl.lam), K, 0.05, 0.01)), orc.hypergrad_fd(prob, wl.w, wl.lam, K, 0.05, 0.01)) < 1e-4
    b.close()


@pytest.mark.parametrize("kind,paired", [("l2", 1), ("l2", 0), ("reweight", 1)])
def test_finite_differences_of_a_large_first_layer(kind, paired, monkeypatch):
    """The first layer's deltas of both points are added before their product with the inputs; ragged tiles."""
    wl = wk.tiny(kind=kind, act="gelu", dims=(1030, 1030, 5), batch=256, hidden=20)
    prob = oracle_problem(wl)
    monkeypatch.setenv("BETTY_TUNE", f"fd2={paired}")
    b = binding.from_workload(wl)
    got = host(b.betty_hypergrad_fd(dev(wl.w), dev(wl.lam), 2, 0.05, 0.01))
    assert rel_l2(got, orc.hypergrad_fd(prob, wl.w, wl.lam, 2, 0.05, 0.01)) < 1e-4
    b.close()
