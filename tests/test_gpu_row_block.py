"""The row-block kernel with its decoder (small THP targets in the layered pass)
against the oracle: verify passes of 17 positions, which the per-sequence pass
leaves to it, over 527 rows (33 tiles of 16, the last ragged), every width in both
precisions, with eight and four waves. Bounds 1e-5 (fp32), 2e-3 (bf16)."""
import dataclasses

import numpy as np
import pytest

from gpu_common import Case, check_verify, gpu_state, histories, weights
from oracle import sampler as S
from oracle.model import Model as OModel
from paper_2507_09252_amd import workloads as W
from test_gpu_prefill import _drafts, _verify

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [8, 4])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("d,F,M,K", [(32, 64, 16, 22), (32, 128, 1, 1), (64, 128, 16, 16), (64, 256, 5, 3)])
def test_row_block_decoder(d, F, M, K, prec, waves, monkeypatch):
    monkeypatch.setenv("TPPSD_BLOCK_NT", str(64 * waves))
    wl = dataclasses.replace(W.WORKLOADS["c2" if prec == "fp32" else "c3"],
                             target=W.ModelCfg(2, d, d // 16, F, M, K, prec),
                             draft=W.ModelCfg(1, 32, 2, 64, M, K, prec), history="hawkes5")
    case = Case(f"{prec}-d{d}-F{F}-M{M}-K{K}", wl, 31, 20, "bias", True, 16)
    print(case.name, waves, flush=True)
    wt, wd = weights(case)
    ht, hk = histories(case)
    hk = hk % K
    dr = _drafts(case, ht, 5)
    want = S.verify(OModel(wl.target, wt), S.prefill(OModel(wl.target, wt), None, ht, hk, 8), dr, np.arange(case.B))
    got = _verify(case, gpu_state(case, wt, wd, case.g, 8, 3), dr, ht, hk, 8)
    check_verify(got, want, 1e-5 if prec == "fp32" else 2e-3, case.name, False, dr)
