"""A paged cache draws, bit for bit, what a contiguous cache of the same rows draws, where both are
scored by the same code: the two-launch step.  The uniforms are placed so that every threshold
whose stratum holds a boundary between two keys lies on that boundary of the float64 CDF, to
float32 rounding: any difference in how the scores round moves some of the draws."""

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2605_01910_amd import santa as S
from tests.gpu_util import KIND_CODE, DeviceWorkload, check_sampled, dev_elems, log, run
from workload import make_workload

pytestmark = pytest.mark.gpu

LENS = [3000, 1777, 17, 2600]


def boundary_uniforms(w):
    """u [B, Hq, S]: (r + u)/S on a boundary of the row's CDF where stratum r holds one."""
    cdf = O.decode_workload(w, "stratified", want_cdf=True).cdf
    u = w.u.copy().reshape(-1, w.S)
    for row in range(u.shape[0]):
        L = int(w.ctx_len[row // w.Hq])
        F = cdf[row, :L - 1]
        for r in range(w.S):
            lo, hi = np.searchsorted(F, [r / w.S, (r + 1) / w.S])
            if hi > lo:
                u[row, r] = np.clip(np.float32(F[(lo + hi) // 2] * w.S - r), 0, np.float32(1 - 2.0 ** -24))
    return u.reshape(w.u.shape)


def contiguous(w, dw):
    """A DeviceWorkload of the same rows in a contiguous cache."""
    c = object.__new__(DeviceWorkload)
    c.w, c.layout, c.q, c.ctx, c.u, c.shape = w, "nhd", dw.q, dw.ctx, dw.u, dw.shape
    for i, name in enumerate(("k", "v")):
        x = np.zeros((w.B, w.n_max, w.Hkv, w.d), w.logical_kv(0)[i].dtype)
        for b in range(w.B):
            x[b, :int(w.ctx_len[b])] = w.logical_kv(b)[i]
        setattr(c, name, dev_elems(x))
    c.kv = S.kv_contiguous(c.k, c.v, c.ctx)
    if w.kv_dtype == "fp8":
        S.set_fp8_cache(c.kv, dw.k_scale, dw.v_scale)
    return c


@pytest.mark.parametrize("G,kv", [(1, "bf16"), (2, "bf16"), (4, "bf16"), (8, "bf16"), (4, "fp8"), (8, "fp8")])
def test_two_launch_draws_of_paged_and_contiguous_caches(G, kv):
    w = make_workload(2, seed=83, paged=True, page_size=16, B=len(LENS), Hkv=2, Hq=2 * G, n=max(LENS), ctx_len=LENS, kind="stratified",
                      S=200, kv_dtype="fp8" if kv == "fp8" else "")
    w.u = boundary_uniforms(w)
    dw = DeviceWorkload(w)
    with S.options("two", splits=4):
        plan = S.santa_plan_info(dw.shape, dw.kv, w.S, KIND_CODE["stratified"])
        assert plan["kernels"] == "k_stream_cdf + k_value_heads", plan
        out, idx, _ = run(w, dw=dw)
        out_c, idx_c, _ = run(w, dw=contiguous(w, dw))
    log(f"[paged equal {kv} G={G}] {int((idx != idx_c).sum())} of {idx.size} draws differ")
    assert np.array_equal(idx, idx_c) and np.array_equal(out, out_c)


@pytest.mark.parametrize("G,B", [(1, 130), (2, 100), (4, 100), (8, 80), (8, 100)])
def test_scheduled_draws_beyond_one_resident_round(G, B):
    """The scheduled step on grids of more workgroups than the matrix-core form holds resident (G =
    8: 640 and 800 of one split a row, where the register form takes one round and two, the other
    two and two): paged and contiguous caches draw the same, and what the oracle draws."""
    lens = [(37 * i) % 200 + 1 for i in range(B - 1)] + [200]
    w = make_workload(2, seed=84, B=B, Hkv=8, Hq=8 * G, n=200, ctx_len=lens, kind="stratified", S=70,
                      paged=True, page_size=16)
    dw = DeviceWorkload(w)
    plan = S.santa_plan_info(dw.shape, dw.kv, w.S, KIND_CODE["stratified"])
    assert (plan["kernels"], plan["splits"]) == ("k_row_sampled", 1), plan
    out, idx, _ = run(w, dw=dw)
    out_c, idx_c, _ = run(w, dw=contiguous(w, dw))
    assert np.array_equal(idx, idx_c) and np.array_equal(out, out_c)
    rows = list(range(0, B * w.Hq, 61))
    log(f"[beyond one round G={G} B={B}] {check_sampled(w, out, idx, rows=rows)}")


def test_scheduled_draws_beyond_two_rounds_of_single_heads():
    """G = 1 on paged caches scores on the matrix cores again beyond 2048 workgroups (2080 of one
    split a row): what the oracle draws."""
    B = 260
    lens = [(37 * i) % 200 + 1 for i in range(B - 1)] + [200]
    w = make_workload(2, seed=85, B=B, Hkv=8, Hq=8, n=200, ctx_len=lens, kind="stratified", S=70,
                      paged=True, page_size=16)
    dw = DeviceWorkload(w)
    plan = S.santa_plan_info(dw.shape, dw.kv, w.S, KIND_CODE["stratified"])
    assert (plan["kernels"], plan["splits"]) == ("k_row_sampled", 1), plan
    out, idx, _ = run(w, dw=dw)
    log(f"[beyond two rounds] {check_sampled(w, out, idx, rows=list(range(0, B * w.Hq, 61)))}")
