"""GPU tests of the decode step (rotation, append, attention, merge of the context's chunks), everything in one launch or
rotation and append in a launch ahead, at the sizes where its parts meet: tile, page, chunk and page-id-window borders, both ways
the metadata reaches the kernel and both ways the chunks are merged."""
import math

import numpy as np
import pytest
import torch

import workloads as W
from oracle import attention as OA
from oracle import rope as R
from paper_2504_19867_amd import semipd as S
from gpu_util import DEV, GpuPool, assert_parity, dev_bf16, f64, host_bits, host_f64

pytestmark = pytest.mark.gpu
DEC = S.SPD_PHASE_DECODE


def _round_bf16(x):
    return f64(W.to_bf16_bits(x))


CASES = [
    # heads, KV heads, dim, page tokens, decode CUs, context lengths, rotary dim (0: no rope), interleaved
    ("tile borders", 8, 2, 128, 16, 128, (1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 64), 128, False),
    ("chunk borders, merged in the launch", 8, 2, 128, 16, 256, (255, 256, 257, 511, 512, 513, 1025), 128, False),
    ("pages of three tiles", 8, 4, 64, 48, 128, (1, 48, 49, 383, 384, 385, 1537, 2600), 32, True),
    ("one query head per KV head, no rope", 4, 4, 64, 16, 128, (1, 130, 700), 0, False),
    ("sixteen query heads per KV head", 16, 1, 128, 64, 256, (33, 900, 1), 64, False),
    ("page ids beyond one window, large pages", 8, 8, 128, 1024, 32, (9001,) * 12, 128, False),
    # at least three workgroups per compute unit, short contexts: records copied, rotation and append by a launch ahead
    ("prepared: tile and page borders", 8, 2, 128, 16, 32, tuple(1 + 31 * i % 68 for i in range(48)), 128, False),
    ("prepared: pages of three tiles, part of the head interleaved", 8, 4, 64, 48, 32, tuple(1 + 29 * i % 131 for i in range(40)), 32, True),
    ("prepared: part of the head, chunks", 4, 4, 128, 32, 32, (1100, 700, 257, 17) * 8, 48, False),
    ("prepared: many query heads", 72, 8, 128, 16, 32, tuple(1 + 7 * i % 40 for i in range(14)), 128, False),
    ("prepared: many KV heads, no rope", 20, 20, 64, 16, 32, tuple(15 + i for i in range(9)), 0, False),
    ("metadata copied, merge launch", 8, 8, 128, 16, 256, tuple(300 + 37 * (i % 29) for i in range(90)), 128, False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_decode_step_appends_rotates_and_attends(case):
    name, H, Hkv, d, P, cus, lens, rot, inter = case
    layer = W.LayerShape("gqa", H, Hkv, d, d, P)
    gp = GpuPool(layer, sum(-(-n // P) for n in lens) + 8, poison=True)       # stale page contents are NaN
    total, _, _ = gp.ctx.device_info()
    gp.ctx.set_partition(total, cus)
    o = R.RopeConfig(theta=500000.0, factor=8.0, rotary_dim=rot, interleaved=inter) if rot else None
    cfg = S.rope_config(theta=500000.0, factor=8.0, rotary_dim=rot, interleaved=inter) if rot else None
    rng = np.random.default_rng(7)
    ids = [10 + i for i in range(len(lens))]
    ks, vs = [], []
    for rid, n in zip(ids, lens):
        k, v = W.normal_bf16(rng, (n, Hkv, d)), W.normal_bf16(rng, (n, Hkv, d))
        gp.pool.kv_reserve(rid, max(n - 1, 1))
        if n > 1:
            gp.pool.kv_write(DEC, rid, 0, n - 1, dev_bf16(k[: n - 1]), dev_bf16(v[: n - 1]))
        ks.append(k)
        vs.append(v)
    gp.ctx.phase_sync(DEC)
    q = W.normal_bf16(rng, (len(lens), H, d))
    scale = 1.0 / math.sqrt(d)
    out = torch.full((len(lens), H, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    tq, tk = dev_bf16(q), dev_bf16(np.stack([k[-1] for k in ks]))
    tv = dev_bf16(np.stack([v[-1] for v in vs]))
    for _ in range(3):                                    # the same step again: counters and workspace are as they were
        gp.pool.decode_step(ids, lens, tq, out, H, scale, k_new=tk, v_new=tv, rope=cfg)
    again = torch.full_like(out, float("nan"))            # and with the token in its page: bit for bit
    gp.pool.decode_step(ids, lens, tq, again, H, scale, rope=cfg)
    gp.ctx.phase_sync(DEC)
    assert np.array_equal(host_bits(out), host_bits(again))
    pos = [n - 1 for n in lens]
    q_rot = _round_bf16(R.apply_rope(f64(q), pos, o)) if rot else f64(q)
    picked = range(len(lens)) if sum(lens) < 20000 else (0, len(lens) // 2, len(lens) - 1)
    for i in picked:
        kk = f64(ks[i])
        if rot:
            kk[-1] = _round_bf16(R.apply_rope(kk[-1:], [pos[i]], o))[0]
        want = OA.decode_attention(q_rot[i], kk, f64(vs[i]), scale)
        assert_parity(host_f64(out[i:i + 1]), want[None], f"{name}: context {lens[i]}")
    gp.close()


def test_steps_past_the_staging_ring_and_pages_freed_behind_them():
    """Many steps without a wait (the staging slots are handed round), then the pages go back while other steps of the
    phase are still queued: a step is known to have finished from the step behind it."""
    layer = W.LayerShape("gqa", 8, 2, 128, 128, 16)
    gp = GpuPool(layer, 64)
    scale = 1.0 / math.sqrt(128)
    rng = np.random.default_rng(8)
    q = dev_bf16(W.normal_bf16(rng, (1, 8, 128)))
    kv = [dev_bf16(W.normal_bf16(rng, (40, 2, 128))) for _ in range(2)]
    outs = [torch.full((1, 8, 128), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(40)]
    for rid in (1, 2):
        gp.pool.kv_reserve(rid, 40)
        gp.pool.kv_write(DEC, rid, 0, 40, kv[0], kv[1])
    for i, o in enumerate(outs):
        gp.pool.decode_step([1 + i % 2], [40], q, o, 8, scale)
    gp.ctx.phase_sync(DEC)
    assert all(np.array_equal(host_bits(o), host_bits(outs[0])) for o in outs)
    gp.pool.decode_step([1], [40], q, outs[0], 8, scale)
    gp.pool.decode_step([2], [40], q, outs[1], 8, scale)
    gp.ctx.phase_sync(DEC)
    gp.pool.kv_free(1)
    gp.pool.kv_free(2)
    gp.close()
