"""The per-sequence verify pass and AR step (one workgroup per sequence) against
the oracle: every width and precision, one to four layers, committed positions
around the 32-key steps and their batches, draft lengths around the 16-position
tile (17 positions take the layered pass), and decoder heads around their
16-row tiles, up to the largest. Bounds as for the workloads of these widths:
1e-5 (fp32), 2e-3 (bf16)."""
import dataclasses

import numpy as np
import pytest

from gpu_common import Case, check_verify, gpu_state, histories, replay_ar_steps, weights
from oracle import sampler as S
from oracle.model import Model as OModel
from paper_2507_09252_amd import workloads as W
from test_gpu_prefill import _drafts, _verify

pytestmark = pytest.mark.gpu


def _case(prec, d, F, L, M, K, n_hist, gamma, B=3):
    base = W.WORKLOADS["c2" if prec == "fp32" else "c3"]
    wl = dataclasses.replace(base, target=W.ModelCfg(L, d, d // 16, F, M, K, prec),
                             draft=W.ModelCfg(1, 32, 2, 64, M, K, prec), history="hawkes5")
    return Case(f"{prec}-d{d}-F{F}-L{L}-M{M}-K{K}-h{n_hist}-g{gamma}", wl, B, n_hist, "bias", True, gamma)


SHAPES = [(p, d, F) for p in ("fp32", "bf16") for d, F in ((32, 64), (32, 128), (64, 128), (64, 256))]
CASES = ([_case(*s, L, 5, 3, 40, 6) for s in SHAPES for L in (1, 4)] +
         # committed positions n_hist - 1: 1, 31 .. 33, several batches per wave
         [_case(p, d, 4 * d, 2, 5, 3, h, 4) for p in ("fp32", "bf16") for d in (32, 64)
          for h in (2, 32, 33, 34, 64, 65, 66, 257, 300)] +
         # 2, 15, 16 and 17 positions
         [_case(p, 64, 256, 2, 5, 3, 50, g) for p in ("fp32", "bf16") for g in (1, 14, 15, 16)] +
         [_case(p, d, 4 * d, 1, M, K, 30, 5) for p, d in (("fp32", 32), ("bf16", 64))
          for M, K in ((1, 1), (16, 17), (17, 16), (33, 1), (64, 64))])


@pytest.mark.parametrize("case", CASES, ids=[c.name for c in CASES])
def test_verify_seq(case):
    wt, wd = weights(case)
    ht, hk = histories(case)
    hk = hk % case.wl.target.n_types
    print(case.name, flush=True)
    dr = _drafts(case, ht, 5)
    T = OModel(case.wl.target, wt)
    want = S.verify(T, S.prefill(T, None, ht, hk, 8), dr, np.arange(case.B))
    got = _verify(case, gpu_state(case, wt, wd, case.g, 8, 3), dr, ht, hk, 8)
    check_verify(got, want, 1e-5 if case.wl.prec == "fp32" else 2e-3, case.name, False, dr)


# (bf16: a draw within 1.1 x 2e-3 of a boundary is a tie and is not compared, so
# that of n components or types about 1 - 4.4e-3 n of the draws are: 0.86 for
# 17 and 16, where 64 and 64 would leave half)
AR_CASES = [_case("fp32", 32, 64, 2, 5, 3, 31, 4), _case("fp32", 64, 256, 4, 5, 3, 31, 4),
            _case("bf16", 64, 128, 2, 5, 3, 31, 4), _case("bf16", 32, 128, 1, 17, 16, 20, 4)]


@pytest.mark.parametrize("case", AR_CASES, ids=[c.name for c in AR_CASES])
def test_ar_step_seq(case):
    from gpu_common import to_dev
    wt, wd = weights(case)
    ht, hk = histories(case)
    hk = hk % case.wl.target.n_types
    case = dataclasses.replace(case, wl=dataclasses.replace(case.wl, name="c2" if case.wl.prec == "fp32" else "c3"))
    st = gpu_state(case, wt, wd, case.g, 12, 9, draft=False)
    st.tppsd_prefill(to_dev(ht), to_dev(hk), 12)
    compared, generated = replay_ar_steps(case, OModel(case.wl.target, wt), st, 9, 12)
    assert st.tppsd_state_status()["bits"] == 0
    assert compared >= 0.5 * generated, (compared, generated)


# which pass serves a job depends on its events, not on the state's capacity: the
# per-sequence pass has no attention launches of its own
@pytest.mark.parametrize("prec,B,n,n_gen,cap,per_seq", [
    ("fp32", 3, 40, 24, 4200, True), ("bf16", 3, 40, 24, 9000, True), ("fp32", 3, 900, 24, 960, False),
    ("bf16", 3, 1900, 24, 1960, False), ("fp32", 3, 380, 600, 1024, False), ("fp32", 80, 900, 24, 960, True)])
def test_pass_follows_the_job(prec, B, n, n_gen, cap, per_seq):
    from gpu_common import to_dev
    from paper_2507_09252_amd import tppsd as tp
    case = _case(prec, 64, 256, 2, 5, 3, n, 4, B)
    wt, wd = weights(case)
    ht, hk = histories(case)
    print(case.name, flush=True)
    st = tp.State(tp.Model(case.wl.target, wt), tp.Model(case.wl.draft, wd), B, cap, 4, seed=1)
    st.tppsd_prefill(to_dev(ht), to_dev(hk % 3), n_gen)
    st.tppsd_timing_enable(tp.TIME_KERNELS)
    st.tppsd_sample_sd(4, max_rounds=2)
    tm = st.tppsd_timing_read()
    st.tppsd_timing_enable(0)
    assert (tm["attn_launches"] == 0) == per_seq, tm
    # the same state, a short job: its graphs are of the other pass
    for job in ((8, 16), (n, n_gen)):
        st.tppsd_prefill(to_dev(ht[:, :job[0]]), to_dev(hk[:, :job[0]] % 3), job[1])
        st.tppsd_sample_sd(4)
        assert st.tppsd_state_status()["n_done"] == B


# n_gen = 0: every sequence is finished. The layered pass fills the caller's rows
# all the same, from the new positions alone; so does the per-sequence pass of the
# widths that both serve (17 positions are the layered pass's)
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_finished_sequences_rows(prec):
    from gpu_common import to_dev
    from paper_2507_09252_amd import tppsd as tp
    case = _case(prec, 64, 256, 2, 5, 3, 40, 16)
    wt, wd = weights(case)
    ht, hk = histories(case)
    dr = _drafts(case, ht, 5)
    rows = []
    for g in (8, 16):
        st = gpu_state(case, wt, wd, g, 8, 3)
        st.tppsd_prefill(to_dev(ht), to_dev(hk % 3), 0)
        dbuf, vbuf = tp.DraftBuffers(case.B, g, 5, 3), tp.VerifyBuffers(case.B, g, 5, 3)
        for dst, src in ((dbuf.tau, dr.tau), (dbuf.t, dr.t), (dbuf.k, dr.k)):
            dst.copy_(to_dev(src[:, :g]))
        vbuf.mix.fill_(float("nan"))
        st.tppsd_verify(g, dbuf, vbuf)
        assert st.tppsd_state_status() == {**st.tppsd_state_status(), "bits": 0, "n_done": case.B}
        rows.append(vbuf.mix[:, :9].cpu().numpy())
    tol = 1e-5 if prec == "fp32" else 2e-3
    assert np.abs(rows[0] - rows[1]).max() <= tol
