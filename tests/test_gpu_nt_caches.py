"""Verify attention with the non-temporal hint: from 384 MiB of keys and values on
(1024 sequences of this target after 800 events) the verify pass has the same bits
as over the first 160 of the sequences alone, whose caches are read plainly."""

import numpy as np
import pytest

from gpu_common import to_dev
from paper_2507_09252_amd import tppsd as tp
from paper_2507_09252_amd import workloads as W

pytestmark = pytest.mark.gpu


# every head width, one and two query tiles
@pytest.mark.parametrize("dh,gamma", [(16, 4), (16, 20), (32, 4), (64, 4)])
def test_nt_reads(dh, gamma):
    B, n, few = 1024, 800, 160
    cfg = W.ModelCfg(2, 64, 64 // dh, 512, 5, 3, "bf16")
    rng = np.random.default_rng(3)
    t = np.cumsum(rng.exponential(size=(B, n + gamma)), 1).astype(np.float32)
    k = rng.integers(0, 3, size=(B, n + gamma)).astype(np.int32)
    model = tp.Model(cfg, W.make_weights(cfg, np.random.SeedSequence(5), "bias"))
    out = []
    for b in (few, B):
        print(dh, gamma, b, flush=True)
        st = tp.State(model, None, b, n + gamma + 9, gamma, seed=1)
        st.tppsd_prefill(to_dev(t[:b, :n]), to_dev(k[:b, :n]), 8)
        dr, v = tp.DraftBuffers(b, gamma, 5, 3), tp.VerifyBuffers(b, gamma, 5, 3)
        dr.tau.copy_(to_dev(np.diff(t[:b, n - 1:], axis=1)))
        dr.t.copy_(to_dev(t[:b, n:]))
        dr.k.copy_(to_dev(k[:b, n:]))
        st.tppsd_verify(gamma, dr, v)
        assert st.tppsd_state_status()["bits"] == 0
        out.append([x[:few].cpu().numpy() for x in (v.logg, v.logf, v.mix, v.logtype)])
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a.view(np.uint32), b.view(np.uint32))
