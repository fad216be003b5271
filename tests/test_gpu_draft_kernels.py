"""The one-launch drafting kernels beside the register kernel, teacher-forced on
their own drafted prefix against the oracle's draft model: one workgroup per
sequence with weights in LDS or global memory (drafts that the register kernel
has no instance for: three and four layers, fp32 of width 64, F = 8 d) and one
wave per sequence (more than 512 sequences, or a few with room for more than 8192
events). Bounds as for the workloads of these widths: 1e-5 (fp32), 2e-3 (bf16)."""
import dataclasses

import numpy as np
import pytest
import torch

from gpu_common import Case, check_draft_record, draft_out, gpu_state, histories, to_dev, weights
from oracle import sampler as S
from oracle.model import Model as OModel
from paper_2507_09252_amd import tppsd as tp
from paper_2507_09252_amd import workloads as W

pytestmark = pytest.mark.gpu


def _case(prec, d, F, L, B=3, n_hist=70, gamma=5, M=5, K=3):
    base = W.WORKLOADS["c2" if prec == "fp32" else "c3"]
    wl = dataclasses.replace(base, target=W.ModelCfg(1, 32, 2, 64, M, K, prec),
                             draft=W.ModelCfg(L, d, d // 16, F, M, K, prec), history="hawkes5")
    return Case(f"{prec}-d{d}-F{F}-L{L}-M{M}-K{K}-h{n_hist}-g{gamma}-B{B}", wl, B, n_hist, "bias", True, gamma)


def _check(case, st, n_gen, rows):
    wt, wd = weights(case)
    ht, hk = histories(case)
    M, K, g = case.wl.target.n_mix, case.wl.target.n_types, case.gamma
    hk = hk % K
    st.tppsd_prefill(to_dev(ht), to_dev(hk), n_gen)
    dbuf = tp.DraftBuffers(case.B, g, M, K)
    st.tppsd_draft(g, dbuf)
    torch.cuda.synchronize()
    assert st.tppsd_state_status()["bits"] == 0
    T, D = OModel(case.wl.target, wt), OModel(case.wl.draft, wd)
    ost = S.prefill(T, D, ht[rows], hk[rows], n_gen)
    tol = 1e-5 if case.wl.prec == "fp32" else 2e-3
    compared = check_draft_record(D, ost, draft_out(dbuf, rows, g), g, 13, 0, rows, tol, case.name)
    assert compared >= 0.9 * len(rows) * g
    # the drafts of one round come from one launch
    st.tppsd_timing_enable(tp.TIME_KERNELS)
    st.tppsd_sample_sd(g, max_rounds=1)
    assert st.tppsd_timing_read()["draft_kernel_launches"] == 1
    st.tppsd_timing_enable(0)


FUSED = ([_case("fp32", 64, F, L) for F in (128, 256) for L in (1, 2)] +
         [_case("fp32", d, 2 * d, 3) for d in (16, 32)] + [_case("fp32", 16, 128, 1), _case("fp32", 32, 256, 2)] +
         [_case("bf16", d, 4 * d, L, M=16, K=22) for d in (32, 64) for L in (3, 4)] +
         [_case("bf16", 32, 256, 1), _case("bf16", 64, 512, 2)] +
         # committed positions around the 64-key steps, several of them; long and short drafts
         [_case(p, 64, 256, L, n_hist=h, gamma=g) for p, L in (("fp32", 1), ("bf16", 3))
          for h, g in ((2, 32), (65, 1), (66, 3), (67, 5), (700, 4))] +
         # more sequences than the LDS form takes
         [_case("bf16", 32, 128, 3, B=257), _case("fp32", 16, 32, 3, B=257)])


@pytest.mark.parametrize("case", FUSED, ids=[c.name for c in FUSED])
def test_draft_one_workgroup(case):
    print(case.name, flush=True)
    wt, wd = weights(case)
    _check(case, gpu_state(case, wt, wd, case.gamma, 40, 13), 40, np.unique(np.linspace(0, case.B - 1, 5).astype(int)))


WAVE = [_case(p, d, f * d, L, B=513, n_hist=40) for p, d in (("fp32", 16), ("fp32", 32), ("bf16", 32)) for f in (2, 4)
        for L in (1, 2)] + [_case("fp32", 32, 128, 1, B=515, n_hist=h, gamma=g) for h, g in ((2, 32), (130, 3))]


@pytest.mark.parametrize("case", WAVE, ids=[c.name for c in WAVE])
def test_draft_one_wave(case):
    print(case.name, flush=True)
    wt, wd = weights(case)
    _check(case, gpu_state(case, wt, wd, case.gamma, 24, 13), 24, np.array([0, 1, 2, 3, 255, 511, case.B - 1]))


@pytest.mark.parametrize("case", [_case(p, 32, 128, 1, B=2) for p in ("fp32", "bf16")], ids=["fp32", "bf16"])
def test_draft_one_wave_long_state(case):
    print(case.name, flush=True)
    wt, wd = weights(case)
    st = tp.State(tp.Model(case.wl.target, wt), tp.Model(case.wl.draft, wd), case.B, 8300, case.gamma, seed=13)
    _check(case, st, 40, np.arange(case.B))
