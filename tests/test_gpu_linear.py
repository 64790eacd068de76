"""The one-workgroup kernel for small single-layer models at the edges of what it takes, against the fp64 oracle."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import betty_oracle as orc
from paper_2207_02849_amd import binding
from paper_2207_02849_amd import workloads as wk
from tests.util import oracle_problem, rel_l2, time_forms

pytestmark = pytest.mark.gpu


# (features and bias in chunks of 32, batches in chunks of 32 and groups of 16 lanes, 1024 threads; whether the series and
# conjugate gradient fit)
@pytest.mark.parametrize("dims,batch,batch_val,loss,bias,fits", [
    ((1, 1), 1, 1, "mse", True, (True, True)),
    ((31, 2), 33, 15, "ce", True, (True, True)),            # 32 entries with the bias
    ((32, 3), 32, 64, "ce", True, (True, True)),            # the bias opens a chunk of its own
    ((64, 1), 512, 256, "mse", False, (True, True)),        # every thread holds data of the validation batch's columns
    ((32, 12), 1024, 1000, "ce", False, (True, True)),      # every thread holds a row; the largest softmax model
    ((1000, 2), 16, 17, "ce", False, (True, True)),         # ... a column
    ((159, 4), 700, 30, "mse", True, (True, False)),        # G at its largest, a train batch the registers could not hold
    ((160, 4), 700, 30, "mse", True, (False, False)),       # ... one more
    ((128, 16), 100, 101, "mse", True, (True, True)),       # operand rows end where the bias begins
])
def test_small_linear_models(dims, batch, batch_val, loss, bias, fits, monkeypatch):
    monkeypatch.setenv("BETTY_TUNE", "linear=1")
    wl = wk.tiny(kind="l2", act="none", dims=dims, batch=max(batch, batch_val), loss=loss, prec="fp32")
    cut = {f: getattr(wl, f)[:n] for f, n in (("X_tr", batch), ("y_tr", batch), ("t_tr", batch), ("X_val", batch_val),
                                              ("y_val", batch_val), ("t_val", batch_val)) if getattr(wl, f) is not None}
    d = dims[0] * dims[1] + (dims[1] if bias else 0)
    wl = dataclasses.replace(wl, has_bias=bias, w=wl.w[:d], lam=wl.lam[:d] + 4.0, **cut)
    prob = oracle_problem(wl)
    b = binding.from_workload(wl)
    w, lam = (torch.as_tensor(np.asarray(a, dtype=np.float32)).cuda() for a in (wl.w, wl.lam))
    for K in (0, 1, 4):
        got = b.betty_hypergrad_neumann(w, lam, K, 0.05).cpu().numpy()
        assert rel_l2(got, orc.hypergrad_neumann(prob, wl.w, wl.lam, K, 0.05)) < 1e-5, ("neumann", K)
        got = b.betty_hypergrad_cg(w, lam, K).cpu().numpy()
        assert rel_l2(got, orc.hypergrad_cg(prob, wl.w, wl.lam, K)) < 1e-4, ("cg", K)
    for call, fit in zip((lambda: b.betty_hypergrad_neumann(w, lam, 4, 0.05), lambda: b.betty_hypergrad_cg(w, lam, 4)), fits):
        b.profile(True)
        call()
        kinds = [r[0] for r in b.profile_records()]
        assert (len(kinds) <= 2 and "shadow" not in kinds) == fit, kinds      # (X^T X and the rest, or launches from the conversion on)
        b.profile(False)
    b.close()


@pytest.mark.parametrize("dims,batch,batch_val,loss,bias,method,K", [
    ((400, 12), 64, 64, "ce", True, "neumann", 2),        # one workgroup 1.9 times the time of the launches
    ((64, 12), 512, 512, "ce", False, "neumann", 1),      # ... 1.6
    ((64, 16), 512, 512, "ce", False, "cg", 1),           # ... 1.9
    ((64, 16), 512, 512, "mse", False, "cg", 1),          # ... 1.6
    ((159, 16), 1024, 128, "mse", True, "neumann", 1),    # ... 1.3
])
def test_one_workgroup_only_where_it_is_the_faster_form(dims, batch, batch_val, loss, bias, method, K, monkeypatch):
    """The rule follows the cost of either form, outputs and steps included."""
    def call(b, w):
        lam = w                                    # (any values: only the time counts)
        return b.betty_hypergrad_cg(w, lam, K) if method == "cg" else b.betty_hypergrad_neumann(w, lam, K, 0.01)
    rule, launches = time_forms(monkeypatch, call, ("", "linear=0"), dims=dims, act="none", loss=loss, hp="l2", prec="fp32",
                                has_bias=bias, batch_train=batch, batch_val=batch_val)
    assert rule < 1.15 * launches, (rule, launches)       # (a few percent between runs)


@pytest.mark.parametrize("dims,batch,bias", [
    ((31, 1), 40, True),                                  # 32 entries: half the registers
    ((32, 2), 40, True),                                  # one more
    ((63, 16), 100, True),                                # 64 entries, an output for every wavefront
    ((64, 17), 33, False),                                # ... and one for a second turn
])
def test_squared_errors_of_few_features(dims, batch, bias, monkeypatch):
    """A wavefront takes an output through all steps by itself; no steps, one, many."""
    wl = wk.tiny(kind="l2", act="none", dims=dims, batch=batch, loss="mse", has_bias=bias)
    prob = oracle_problem(wl)
    monkeypatch.setenv("BETTY_TUNE", "linear=1")
    b = binding.from_workload(wl)
    for K in (0, 1, 20):
        got = b.betty_hypergrad_neumann(torch.as_tensor(wl.w).cuda(), torch.as_tensor(wl.lam).cuda(), K, 0.02).cpu().numpy()
        assert rel_l2(got, orc.hypergrad_neumann(prob, wl.w, wl.lam, K, 0.02)) < 1e-5, K
    b.close()


def test_squared_errors_of_few_features_take_no_longer_than_many(monkeypatch):
    """A single step: what the form of up to 64 features sets up is no more than what it saves (9.7 against 8.9 us when every
    wavefront did, beside one output)."""
    call = lambda b, w: b.betty_hypergrad_neumann(w, w, 1, 1e-4)
    ratios = []
    for _ in range(9):                                    # (close together: the card's speed changes now and then)
        few, many = (time_forms(monkeypatch, call, ("linear=1",), rounds=3, dims=(n, 1), act="none", loss="mse", hp="l2", prec="fp32",
                                has_bias=True, batch_train=200, batch_val=100)[0] for n in (7, 64))
        ratios.append(few / many)
    assert np.median(ratios) < 1.0, ratios
