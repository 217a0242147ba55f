"""The sampled steps' matrix-core score stage (ring_scores) at the edges of its 16-key tiles and
splits, against the CPU oracle: rows of 0 keys, of one key, of a tile plus or minus one, fewer
tiles than waves, splits longer than the ring; pages of 4 to 64 keys, and groups of eight query
heads on every cache.  What lies past a row's length is NaN: none of it may reach the output.
The products of a key are the same as on the vector units and their sums round no worse
(test_gpu_score_rounding.py), so the indices keep the oracle's 1e-5 band."""

import numpy as np
import pytest
import torch

from paper_2605_01910_amd import santa as S
from tests.gpu_util import DeviceWorkload, KIND_CODE, check_sampled, current_rows, log, run
from tests.test_gpu_dense_stream import _poison
from workload import make_workload

pytestmark = pytest.mark.gpu

LENS = [0, 1, 15, 16, 17, 63, 65, 1023, 1024, 1025, 2600]


@pytest.mark.parametrize("kind", ["systematic", "stratified"])
@pytest.mark.parametrize("path,kernels", [("rows", "k_row_sampled"), ("two", "k_stream_cdf")])
@pytest.mark.parametrize("cache,G", [("page4", 4), ("page16", 1), ("page16", 2), ("page16", 4), ("page64", 4),
                                     ("page4", 8), ("page16", 8), ("bf16", 8), ("fp8", 8), ("fp8page16", 8)])
def test_ring_scores_edges(cache, G, path, kernels, kind):
    over = dict(B=len(LENS), Hkv=2, Hq=2 * G, n=max(LENS), ctx_len=LENS, kind=kind, S=40)
    if cache.startswith("fp8"):
        over["kv_dtype"] = "fp8"
    if "page" in cache:
        over.update(paged=True, page_size=int(cache.split("page")[1]))
    w = make_workload(2, seed=79, **over)
    dw = DeviceWorkload(w)
    _poison(dw, w)
    with S.options(path, splits=3):
        plan = S.santa_plan_info(dw.shape, dw.kv, w.S, KIND_CODE[kind])
        assert kernels in plan["kernels"], plan
        out, idx, _ = run(w, dw=dw)
        again, idx2, _ = run(w, dw=dw)
    assert np.array_equal(out, again) and np.array_equal(idx, idx2)
    log(f"[ring scores {cache} G={G} {path} {kind}] {check_sampled(w, out, idx)}")


@pytest.mark.parametrize("S_", [65, 129, 1000])
@pytest.mark.parametrize("cache", ["bf16", "page16", "fp8"])
def test_more_claims_than_lanes(cache, S_):
    """Groups of eight, stratified: a split that takes more than 64 claims of a head goes through
    several passes, each fetching the next one's uniforms.  The row of 40 keys takes all S in one
    split; 65 and 129 leave one claim to the last pass."""
    over = dict(B=4, Hkv=2, Hq=16, n=2600, ctx_len=[0, 40, 700, 2600], kind="stratified", S=S_)
    if cache == "fp8":
        over["kv_dtype"] = "fp8"
    if cache == "page16":
        over.update(paged=True, page_size=16)
    w = make_workload(2, seed=80, **over)
    dw = DeviceWorkload(w)
    _poison(dw, w)
    with S.options("rows", splits=3):
        plan = S.santa_plan_info(dw.shape, dw.kv, w.S, KIND_CODE["stratified"])
        assert plan["kernels"] == "k_row_sampled", plan
        out, idx, _ = run(w, dw=dw)
    log(f"[claims {cache} S={S_}] {check_sampled(w, out, idx)}")


APPEND_LENS = [1, 16, 17, 64, 65, 1024, 1025, 2600]  # the last key: alone, last or first of a tile, of a split


@pytest.mark.parametrize("path", ["rows", "two"])
@pytest.mark.parametrize("cache,G", [("bf16", 8), ("page4", 8), ("page16", 8), ("page16", 4)])
def test_ring_scores_append(cache, G, path):
    """The current token's rows, stored by the call and then copied into the ring: the cache holds
    NaN there before, and past it."""
    over = dict(B=len(APPEND_LENS), Hkv=2, Hq=2 * G, n=max(APPEND_LENS), ctx_len=APPEND_LENS,
                kind="stratified", S=100)
    if "page" in cache:
        over.update(paged=True, page_size=int(cache.split("page")[1]))
    w = make_workload(2, seed=86, **over)
    dw = DeviceWorkload(w)
    rows = current_rows(dw, w)
    k_new = torch.stack([k.clone() for k, _ in rows]).contiguous()
    v_new = torch.stack([v.clone() for _, v in rows]).contiguous()
    _poison(dw, w)
    for k, v in rows:
        k.fill_(float("nan"))
        v.fill_(float("nan"))
    dw.kv.k_new, dw.kv.v_new = k_new.data_ptr(), v_new.data_ptr()
    with S.options(path, splits=3):
        out, idx, _ = run(w, dw=dw)
    for b, (k, v) in enumerate(rows):
        assert torch.equal(k, k_new[b]) and torch.equal(v, v_new[b]), f"cache row of sequence {b}"
    log(f"[ring append {cache} G={G} {path}] {check_sampled(w, out, idx)}")
