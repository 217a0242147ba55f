"""The streaming dense kernel (k_dense_stream) at the edges of its tiles and splits, against the
CPU oracle: rows of 0 keys, of one key, of 16-key tiles plus or minus one, splits shorter than
four tiles (waves without a tile), every group size and element type, pages of 4 to 64 keys.
What lies past a row's length in the cache is NaN: none of it may reach the output."""

import numpy as np
import pytest
import torch

from paper_2605_01910_amd import santa as S
from tests.gpu_util import DeviceWorkload, check_dense, current_rows, log, run
from workload import make_workload

pytestmark = pytest.mark.gpu

SHORT = [0, 1, 15, 16, 17, 63, 64, 65, 500]          # splits of 64 keys
LONG = [0, 1, 255, 256, 257, 700, 1025, 2599, 2600]  # splits of 256 keys


def _poison(dw, w):
    """NaN in every cache row at or past a sequence's length (FP8: the NaN code)."""
    bad = 0x7F if w.kv_dtype == "fp8" else float("nan")
    for b, L in enumerate(w.ctx_len.tolist()):
        if w.paged:
            first, ps = -(-L // w.page_size), w.page_size
            if L % ps:
                page = int(w.block_table[b, first - 1])
                for t in (dw.kp, dw.vp):
                    t[page, :, L % ps:] = bad
        else:
            for t in (dw.k, dw.v):
                t[b, L:] = bad


@pytest.mark.parametrize("lens", [SHORT, LONG], ids=["short", "long"])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("cache", ["bf16", "fp8", "page4", "page16", "page64"])
def test_dense_stream_edges(cache, G, lens):
    Hkv, n = 8, max(lens)
    over = dict(B=len(lens), Hkv=Hkv, Hq=Hkv * G, n=n, ctx_len=lens, kind="systematic", S=16)
    if cache == "fp8":
        over["kv_dtype"] = "fp8"
    if cache.startswith("page"):
        over.update(paged=True, page_size=int(cache[4:]))
    w = make_workload(2, seed=77, **over)
    dw = DeviceWorkload(w)
    _poison(dw, w)
    with S.options("auto", splits=8 if lens is SHORT else 12):  # 72 rows x 8 or 11 splits
        plan = S.santa_plan_info(dw.shape, dw.kv, 1, S.SANTA_KIND_DENSE)
        assert plan["kernels"] == "k_dense_stream", plan
        out, _, _ = run(w, "dense", dw=dw)
        again, _, _ = run(w, "dense", dw=dw)
    assert np.array_equal(out, again)
    assert np.all(out[: w.Hq] == 0)  # the empty row
    log(f"[dense stream {cache} G={G}] {check_dense(w, out)}")


def test_dense_stream_scores_of_minus_infinity():
    """A split whose keys all score -inf weighs nothing; the others' keys keep their weights."""
    w = make_workload(2, seed=78, B=9, Hkv=8, Hq=32, n=512, kind="systematic", S=16)
    dw = DeviceWorkload(w)
    with S.options("auto", splits=8):
        assert S.santa_plan_info(dw.shape, dw.kv, 1, S.SANTA_KIND_DENSE)["kernels"] == "k_dense_stream"
        ref, _, _ = run(w, "dense", dw=dw)
        k = dw.k.clone()
        dw.q[..., 0] = 1.0               # one positive feature for every head
        dw.k[:, 64:128, :, 0] = float("-inf")
        out, _, _ = run(w, "dense", dw=dw)
    keep = torch.ones(512, dtype=torch.bool)
    keep[64:128] = False
    q, k, v = (t.double().cpu() for t in (dw.q, k, dw.v))
    s = torch.einsum("bkgd,bnkd->bkgn", q.view(9, 8, 4, 128), k[:, keep]) * w.scale
    o = torch.einsum("bkgn,bnkd->bkgd", torch.softmax(s, -1), v[:, keep]).reshape(-1, 128).numpy()
    assert np.all(np.isfinite(ref)) and np.abs(out - o).max() <= 2e-2


# the last key: the only one, the last or first of a tile, of a split of 64 (128, 320) keys, neither
APPEND_SHORT = [1, 16, 17, 64, 65, 129, 449, 490, 500]
APPEND_LONG = [1, 128, 129, 256, 257, 700, 1025, 2561, 2600]


@pytest.mark.parametrize("lens", [APPEND_SHORT, APPEND_LONG], ids=["short", "long"])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("cache", ["nhd", "hnd", "page4", "page16", "page64"])
def test_dense_stream_append(cache, G, lens):
    """The current token's rows, stored by the call and then read through LDS copies: the cache holds
    NaN there before, and past it.  Head-major and sequence-major caches and pages."""
    Hkv, n = 8, max(lens)
    over = dict(B=len(lens), Hkv=Hkv, Hq=Hkv * G, n=n, ctx_len=lens, kind="systematic", S=16)
    if cache.startswith("page"):
        over.update(paged=True, page_size=int(cache[4:]))
    w = make_workload(2, seed=85, **over)
    dw = DeviceWorkload(w, "hnd" if cache == "hnd" else "nhd")
    rows = current_rows(dw, w)
    k_new = torch.stack([k.clone() for k, _ in rows]).contiguous()
    v_new = torch.stack([v.clone() for _, v in rows]).contiguous()
    if cache == "hnd":
        for b, L in enumerate(lens):
            dw.k[b, :, L:] = dw.v[b, :, L:] = float("nan")
    else:
        _poison(dw, w)
    kinds = {}
    for append in (False, True):
        if append:
            for k, v in rows:
                k.fill_(float("nan"))
                v.fill_(float("nan"))
            dw.kv.k_new, dw.kv.v_new = k_new.data_ptr(), v_new.data_ptr()
        with S.options("auto", splits=8 if lens is APPEND_SHORT else 12):
            plan = S.santa_plan_info(dw.shape, dw.kv, 1, S.SANTA_KIND_DENSE)
            assert plan["kernels"] == "k_dense_stream", plan
            kinds[append], _, _ = run(w, "dense", dw=dw)
    for b, (k, v) in enumerate(rows):
        assert torch.equal(k, k_new[b]) and torch.equal(v, v_new[b]), f"cache row of sequence {b}"
    assert np.array_equal(kinds[False], kinds[True])
    log(f"[dense stream append {cache} G={G}] {check_dense(w, kinds[True])}")
