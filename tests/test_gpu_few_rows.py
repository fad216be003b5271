"""The few-row GEMM (16 x 16 tiles) through verify
passes of B (gamma + 1) rows at the edges of its tiles and of its row limits,
against the oracle, with the fixed per-workload bounds of gpu_common. The
products of these targets take every instance: K of 4, 8, 16, 32 and 64
k-steps, with and without a LayerNorm operand, in bf16 and fp32, and a head
product whose columns are no multiple of 16."""
import dataclasses

import numpy as np
import pytest

from gpu_common import Case, check_verify, gpu_state, histories, small, to_dev, tol_of, weights
from oracle import sampler as S
from oracle.model import Model as OModel
from paper_2507_09252_amd import workloads as W
from test_gpu_prefill import _drafts, _verify

pytestmark = pytest.mark.gpu

# fp32 of width 128 and 256 (8 and 16 k-steps, FFN and head products of 16, 32 and 64)
F128 = dataclasses.replace(W.WORKLOADS["c2"], target=W.ModelCfg(1, 128, 4, 256, 5, 3, "fp32"),
                           draft=W.ModelCfg(1, 32, 2, 64, 5, 3, "fp32"), history="hawkes5")
F256 = dataclasses.replace(F128, target=W.ModelCfg(1, 256, 4, 1024, 5, 3, "fp32"))


def _rows(name, wl, B, gamma):
    return Case(f"{name}-T{B * (gamma + 1)}", wl, B, 20, "bias", True, gamma)


CASES = [_rows(n, W.WORKLOADS[n], B, g) for n, B, g in
         [("c4", 1, 1), ("c4", 3, 4), ("c4", 2, 7), ("c4", 1, 16), ("c4", 14, 7), ("c4", 38, 2), ("c4", 16, 7),
          ("c4", 43, 2),
          ("c3", 1, 14), ("c3", 16, 7), ("c3", 43, 2), ("c3", 32, 7), ("c3", 43, 5),
          ("c2", 1, 1), ("c2", 3, 10), ("c2", 32, 7), ("c2", 43, 5),
          ("a3", 1, 6), ("a3", 16, 7), ("a3", 43, 2), ("c5", 5, 8), ("c5", 8, 7), ("c5", 32, 7)]] + [
    _rows("f128", F128, 3, 5), _rows("f128", F128, 32, 7), _rows("f256", F256, 7, 4), _rows("f256", F256, 43, 5)]


@pytest.mark.parametrize("case", CASES, ids=[c.name for c in CASES])
def test_verify_few_rows(case):
    wt, wd = weights(case)
    ht, hk = histories(case)
    hk = hk % case.wl.target.n_types
    print(f"{case.name}: B {case.B}, gamma {case.g}", flush=True)
    dr = _drafts(case, ht, 5)
    want = S.verify(OModel(case.wl.target, wt), S.prefill(OModel(case.wl.target, wt), None, ht, hk, 8), dr,
                    np.arange(case.B))
    got = _verify(case, gpu_state(case, wt, wd, case.g, 8, 3), dr, ht, hk, 8)
    check_verify(got, want, tol_of(case.wl), case.name, False, dr)


# a step's events have the same bits whatever the batch: rows in the few-row
# GEMM's tiles and (from 113 or 257 rows) in the staged ones
@pytest.mark.parametrize("name,B", [("c4", 17), ("c3", 17), ("a3", 17), ("c5", 17), ("c5", 96)])
def test_step_bits_do_not_depend_on_batch(name, B):
    wl = W.WORKLOADS[name]
    big = Case("batch", wl, 300, 2, "bias", True, 1)
    wt, wd = weights(big)
    ht, hk = histories(big)
    print(f"{name}: B {B} and {big.B}", flush=True)
    runs = []
    for b in (B, big.B):
        case = dataclasses.replace(big, B=b)
        st = gpu_state(case, wt, wd, 1, 24, 7, draft=False)
        st.tppsd_prefill(to_dev(ht[:b]), to_dev(hk[:b]), 24)
        st.tppsd_sample_ar(24)
        t, k, _ = st.tppsd_read_events()
        runs.append((t[:B, :26].cpu().numpy().view(np.uint32), k[:B, :26].cpu().numpy()))
    assert np.array_equal(runs[0][0], runs[1][0]) and np.array_equal(runs[0][1], runs[1][1])
