"""Drafting with the model in registers, teacher-forced on its own drafted
prefix against the oracle's draft model: every instance of the kernel (widths,
FFN widths, one and two layers, both precisions, both encoders), committed
positions around the 64-key steps and the batches of them (and none at all),
head counts around their 16-row tiles, and draft lengths from 1 to 32. Bounds:
1e-5 (fp32) and 2e-3 (bf16) on the recorded distributions, as for the workloads
of these widths; draws, densities and types as in gpu_common."""
import dataclasses

import numpy as np
import pytest
import torch

from gpu_common import Case, check_draft_record, draft_out, gpu_state, histories, to_dev, tol_of, weights
from oracle import sampler as S
from oracle.model import Model as OModel
from paper_2507_09252_amd import tppsd as tp
from paper_2507_09252_amd import workloads as W

pytestmark = pytest.mark.gpu


def _case(prec, d, f, L, M, K, n_hist, gamma, enc="thp", B=3):
    base = W.WORKLOADS["c2" if prec == "fp32" else "c3"]
    t = W.ModelCfg(1, 32, 2, 64, M, K, prec, enc, 0.1, 50.0)
    wl = dataclasses.replace(base, target=t, draft=W.ModelCfg(L, d, d // 16, f * d, M, K, prec, enc, 0.1, 50.0),
                             history="hawkes5")
    return Case(f"{enc}-{prec}-d{d}-F{f * d}-L{L}-M{M}-K{K}-h{n_hist}-g{gamma}-B{B}", wl, B, n_hist, "bias", True, gamma)


CASES = (
    [_case("fp32", d, f, L, 5, 3, 70, 6) for d in (16, 32) for f in (2, 4) for L in (1, 2)] +
    [_case("bf16", d, f, L, 16, 22, 70, 6) for d in (32, 64) for f in (2, 4) for L in (1, 2)] +
    [_case(p, d, 0, L, 5, 3, 70, 6, "attnhp") for p, ds in (("fp32", (16, 32)), ("bf16", (32, 64))) for d in ds
     for L in (1, 2)] +
    # committed positions (n_hist - 2): none, 1, whole and ragged 64-key steps,
    # several batches per wave; the longest and shortest drafts
    [_case(p, d, f, L, 5, 3, h, g) for p, d, f, L in (("fp32", 16, 2, 1), ("fp32", 32, 4, 1), ("bf16", 64, 4, 2))
     for h, g in ((2, 1), (2, 32), (3, 5), (65, 2), (66, 3), (67, 32), (130, 2), (700, 4))] +
    [_case("bf16", 64, 0, 2, 16, 22, h, g, "attnhp") for h, g in ((2, 32), (66, 2), (700, 4))] +
    # decoder heads: rows around the 16-row tiles
    [_case("bf16", 32, 4, 1, M, K, 40, 4) for M, K in ((1, 1), (15, 17), (16, 16), (17, 1), (32, 32))] +
    [_case("fp32", 32, 4, 1, M, K, 40, 4) for M, K in ((1, 16), (17, 31))])


@pytest.mark.parametrize("case", CASES, ids=[c.name for c in CASES])
def test_draft_regs(case):
    wt, wd = weights(case)
    ht, hk = histories(case)
    M, K, g, seed, n_gen = case.wl.target.n_mix, case.wl.target.n_types, case.gamma, 13, 40
    hk = hk % K
    print(case.name, flush=True)
    T, D = OModel(case.wl.target, wt), OModel(case.wl.draft, wd)
    st = gpu_state(case, wt, wd, g, n_gen, seed)
    st.tppsd_prefill(to_dev(ht), to_dev(hk), n_gen)
    dbuf = tp.DraftBuffers(case.B, g, M, K)
    st.tppsd_draft(g, dbuf)
    torch.cuda.synchronize()
    assert st.tppsd_state_status()["bits"] == 0
    rows = np.arange(case.B)
    ost = S.prefill(T, D, ht, hk, n_gen)
    tol = 1e-5 if case.wl.prec == "fp32" else 2e-3
    compared = check_draft_record(D, ost, draft_out(dbuf, rows, g), g, seed, 0, rows, tol, case.name)
    assert compared >= 0.9 * case.B * g


# THP's attention probabilities stay in fp32: the mixtures of the first draft
# agree with the wave-per-sequence kernel's, which serves the next larger batch,
# to the last bits of the sums and a few 16-bit roundings of activations that
# these tip (measured 5.5e-8 and 8.1e-8, relative 2-norm; with probabilities
# rounded to bf16, as many roundings as keys, 3.2e-6)
def test_draft_probabilities_are_not_rounded():
    wl = W.WORKLOADS["c5"]
    ht, hk = W.make_histories(wl, batch=513, n_hist=200)
    wt, wd = W.workload_weights(wl, init="bias")
    M, K, out = wl.target.n_mix, wl.target.n_types, []
    for B in (512, 513):
        st = tp.State(tp.Model(wl.target, wt), tp.Model(wl.draft, wd), B, 260, 4, seed=1)
        st.tppsd_prefill(to_dev(ht[:B]), to_dev(hk[:B]), 50)
        buf = tp.DraftBuffers(B, 4, M, K)
        st.tppsd_draft(4, buf)
        out.append([x[:512, 0].double().cpu() for x in (buf.mix, buf.logtype)])
    for a, b in zip(*out):
        assert (a - b).norm() / a.norm() < 1e-6
