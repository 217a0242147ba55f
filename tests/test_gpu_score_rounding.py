"""Rounding error of the scores, seen through the dense step.  Two keys whose exact scores are
equal -- the query's magnitudes come in 16 classes of 8 features, and the second key is the first
with its features permuted within each class and signed accordingly -- differ after rounding by e,
and with values 1 and 0 and a softmax scale of 2^20 ln 2 the output is 1 / (1 + 2^-(2^20 e)), from
which e is read back to the 8 bits of a bfloat16.  Grids above 512 workgroups take the matrix-core
score stage (k_dense_stream), grids of 256 the vector-unit one (k_fused_dense): the first may not
round worse than the second."""

import math

import pytest
import torch

from paper_2605_01910_amd import santa as S
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

D, HKV, ROWS = 128, 8, 4096   # rows: (sequence, KV head) pairs, one score difference each
SCALE = 2.0 ** 20 * math.log(2.0)


def _differences(q, kv_of, B, kernel):
    """2^20 (s_0 - s_1) of every row, from dense steps over B sequences at a time."""
    out = torch.empty_like(q)
    for b in range(0, q.shape[0], B):
        kv, shape = kv_of(b, B), S.shape_of(q[b:b + B], HKV)
        assert S.santa_plan_info(shape, kv, 1, S.SANTA_KIND_DENSE)["kernels"] == kernel
        ws = S.alloc_workspace(shape, kv, 1, S.SANTA_KIND_DENSE)
        S.santa_decode_dense(q[b:b + B], kv, shape, SCALE, out[b:b + B], ws)
        torch.cuda.synchronize()
    p = out[:, ::q.shape[1] // HKV, 0].double().clamp(2.0 ** -8, 1 - 2.0 ** -8)
    return torch.log2(p / (1 - p))


@pytest.mark.parametrize("cache,G", [("bf16", 2), ("bf16", 4), ("bf16", 8), ("fp8", 4)])
def test_matrix_core_scores_round_no_worse_than_vector_scores(cache, G):
    g = torch.Generator(device="cuda").manual_seed(5)
    n_seq = ROWS // HKV
    rms = {}
    for _ in range(4):
        sign = torch.randint(0, 2, (n_seq, HKV, D), generator=g, device="cuda") * 2.0 - 1.0
        place = torch.rand(n_seq, HKV, D, generator=g, device="cuda").argsort(-1)  # class = rank // 8
        mag = (torch.rand(n_seq, HKV, D // 8, generator=g, device="cuda") + 0.5).bfloat16().float()
        mag = torch.empty_like(sign).scatter_(-1, place, mag.repeat_interleave(8, -1))
        a = torch.randn(n_seq, HKV, D, generator=g, device="cuda")
        a = (a * 8).to(torch.float8_e4m3fn).float() / 8 if cache == "fp8" else a.bfloat16().float()
        # feature place[r] of the second key comes from place[r'], r' another rank of r's class
        shuffle = torch.rand(n_seq, HKV, D // 8, 8, generator=g, device="cuda").argsort(-1)
        shuffle = (shuffle + 8 * torch.arange(D // 8, device="cuda")[:, None]).flatten(-2)
        perm = torch.empty_like(place).scatter_(-1, place, place.gather(-1, shuffle))
        k = torch.stack([a, a.gather(-1, perm) * sign.gather(-1, perm) * sign], 1)   # [B, 2, Hkv, D]
        v = torch.stack([torch.ones_like(a), torch.zeros_like(a)], 1)
        if cache == "fp8":
            k, v = ((t * 8).to(torch.float8_e4m3fn).view(torch.uint8) for t in (k, v))
            scale = torch.full((n_seq, HKV), 0.125, device="cuda")
        else:
            k, v = k.bfloat16(), v.bfloat16()
        q = (sign * mag).bfloat16().repeat_interleave(G, 1)

        def kv_of(b, B):
            kv = S.kv_contiguous(k[b:b + B], v[b:b + B])
            if cache == "fp8":
                S.set_fp8_cache(kv, scale[b:b + B], scale[b:b + B])
            return kv

        for B, kernel in ((n_seq, "k_dense_stream"), (32, "k_fused_dense")):
            e = _differences(q, kv_of, B, kernel)
            rms.setdefault(kernel, []).append(e.square().mean())
    new, old = (math.sqrt(torch.stack(rms[n]).mean().item()) for n in ("k_dense_stream", "k_fused_dense"))
    log(f"[score rounding {cache} G={G}] matrix cores {new:.4f}, vector units {old:.4f} (units of 2^-20)")
    # 16384 differences each: the ratio of their rms is known to about 1 %, and 4 % is four deviations
    assert 0 < new <= 1.04 * old
