"""The fused layer kernel through verify passes of B (gamma + 1) rows, against
the oracle, with the fixed per-workload bounds of gpu_common: d = 128 (48-row
tiles) at a few rows and from 8192, d = 256 in 16-row tiles up to 4096 rows and
in 32-row tiles above, ragged and whole last tiles, and head widths of 16, 32
and 64 (the order in which keys and values are stored)."""
import dataclasses

import numpy as np
import pytest

from gpu_common import Case, check_verify, gpu_state, histories, tol_of, weights
from oracle import sampler as S
from oracle.model import Model as OModel
from paper_2507_09252_amd import workloads as W
from test_gpu_prefill import _drafts, _verify

pytestmark = pytest.mark.gpu


def _wl(d, H, F):
    return dataclasses.replace(W.WORKLOADS["c5"], target=W.ModelCfg(2, d, H, F, 16, 5, "bf16"),
                               draft=W.ModelCfg(1, 32, 2, 64, 16, 5, "bf16"), history="hawkes5")


CASES = [Case(f"d{d}-H{H}-T{B * (g + 1)}", _wl(d, H, F), B, 20, "bias", True, g) for d, H, F, B, g in
         [(128, 4, 512, 1, 2), (128, 8, 512, 12, 3), (128, 2, 512, 16, 3), (128, 4, 512, 911, 8), (128, 8, 512, 1024, 8),
          (256, 8, 1024, 187, 10), (256, 16, 1024, 256, 15), (256, 4, 1024, 241, 16), (256, 8, 1024, 288, 15)]]


@pytest.mark.parametrize("case", CASES, ids=[c.name for c in CASES])
def test_verify_layer_rows(case, monkeypatch):
    monkeypatch.setenv("TPPSD_FFN_FUSED", "1")   # (a few rows run the few-row products by default)
    wt, wd = weights(case)
    ht, hk = histories(case)
    hk = hk % case.wl.target.n_types
    print(f"{case.name}: B {case.B}, gamma {case.g}", flush=True)
    dr = _drafts(case, ht, 5)
    want = S.verify(OModel(case.wl.target, wt), S.prefill(OModel(case.wl.target, wt), None, ht, hk, 8), dr,
                    np.arange(case.B))
    got = _verify(case, gpu_state(case, wt, wd, case.g, 8, 3), dr, ht, hk, 8)
    check_verify(got, want, tol_of(case.wl), case.name, False, dr)
