"""The launch that carries a prefill step's rows (page write, rotation of keys and queries), in plain and in chunked steps:
the sizes where its tiles, head groups and pieces end, against the same work done call by call (bit for bit: copies, and one
rotation arithmetic) and the fp64 oracle's attention."""
import math

import numpy as np
import pytest
import torch

import workloads as W
from oracle import attention as OA
from paper_2504_19867_amd import semipd as S
from gpu_util import DEV, GpuPool, assert_parity, dev_bf16, f64, host_bits, host_f64

pytestmark = pytest.mark.gpu
PRE = S.SPD_PHASE_PREFILL

CASES = [
    # q heads, KV heads, dim, rotating entries, their offset, interleaved, new rows, cached rows
    (4, 2, 64, 64, 0, False, (1, 16, 17), (15, 16, 17)),               # fewer heads than a group
    (18, 9, 128, 128, 0, False, (31, 2), (1, 33)),                     # a second group of KV heads, and a third of query heads, with a remainder
    (10, 2, 128, 48, 16, False, (15, 40), (0, 3)),                     # part of the head, a request without a prefix
    (8, 8, 64, 16, 48, True, (5, 64), (63, 1)),                        # one piece pair per head
    (16, 8, 128, 96, 32, True, (33,), (47,)),
    (64, 8, 128, 128, 0, False, (2060, 5), (0, 21)),                   # queries in a launch of their own (more than 32 MiB of them)
]


@pytest.mark.parametrize("rope", (False, True), ids=("plain", "rope"))
@pytest.mark.parametrize("H,Hkv,d,rot,off,inter,lens,pre", CASES)
def test_rows_of_a_chunked_step(H, Hkv, d, rot, off, inter, lens, pre, rope):
    layer = W.LayerShape("gqa", H, Hkv, d, d, 16)
    ids, scale = list(range(1, len(lens) + 1)), 1.0 / math.sqrt(d)
    q, k, v, cu = W.prefill_inputs(layer, lens, seed=7 + H + d)
    cfg = S.rope_config(theta=10000.0, rotary_dim=rot, rotary_offset=off, interleaved=inter) if rope else None
    gp = GpuPool(layer, sum(-(-(n + p) // 16) for n, p in zip(lens, pre)) + 2, poison=True)
    cached = [(W.normal_bf16(np.random.default_rng(100 + r), (p, Hkv, d)), W.normal_bf16(np.random.default_rng(200 + r), (p, Hkv, d)))
              for r, p in zip(ids, pre)]
    for r, p, (kc, vc) in zip(ids, pre, cached):
        if p:
            gp.pool.kv_reserve(r, p)
            gp.pool.kv_write(PRE, r, 0, p, dev_bf16(kc), dev_bf16(vc))
    tq, tk, tv = dev_bf16(q), dev_bf16(k), dev_bf16(v)
    wq, wk = dev_bf16(q), dev_bf16(k)
    if rope:
        pos = np.concatenate([p + np.arange(n) for p, n in zip(pre, lens)])
        gp.ctx.rope_qk(PRE, cfg, [int(x) for x in pos], wq, H, wk, Hkv, d)
    out = torch.empty((cu[-1], H, d), dtype=torch.bfloat16, device=DEV)
    gp.pool.prefill_step(ids, cu, tq, tk, tv, out, H, Hkv, d, d, scale, prefix_lens=list(pre), rope=cfg)
    gp.ctx.phase_sync(PRE)
    np.testing.assert_array_equal(host_bits(tq), host_bits(wq))
    np.testing.assert_array_equal(host_bits(tk), host_bits(wk))
    q_bits, k_bits, got = host_bits(wq), host_bits(wk), host_f64(out)
    for i, (r, p, n) in enumerate(zip(ids, pre, lens)):
        kg = torch.empty((p + n, Hkv, d), dtype=torch.bfloat16, device=DEV)
        vg = torch.empty_like(kg)
        gp.pool.kv_gather(PRE, r, p + n, kg, vg)
        gp.ctx.phase_sync(PRE)
        k_all, v_all = np.concatenate([cached[i][0], k_bits[cu[i]:cu[i + 1]]]), np.concatenate([cached[i][1], v[cu[i]:cu[i + 1]]])
        np.testing.assert_array_equal(host_bits(kg), k_all)
        np.testing.assert_array_equal(host_bits(vg), v_all)
        a = max(0, n - 64)                           # the oracle takes the last rows: they see all the others
        want = OA.chunk_attention(f64(q_bits[cu[i] + a:cu[i + 1]]), f64(k_all), f64(v_all), scale)
        assert_parity(got[cu[i] + a:cu[i + 1]], want, f"request {i}")
    gp.close()


@pytest.mark.parametrize("rope", (False, True), ids=("plain", "rope"))
@pytest.mark.parametrize("H,Hkv,d", [(8, 8, 128), (5, 5, 64), (18, 9, 128)])
@pytest.mark.parametrize("tiles", [1, 8, 9, 16, 17, 31, 32, 33, 64, 65])
def test_rows_by_any_number_of_heads_per_workgroup(tiles, H, Hkv, d, rope):
    """One, two, four or eight KV heads per workgroup, by tiles against the share's 32 compute units (twice as many with nine heads, whose
    workgroups of eight are two per tile): both sides of every change, head counts with a remainder of each group."""
    layer = W.LayerShape("gqa", H, Hkv, d, d, 16)
    lens = (16 * tiles - 5,) if tiles < 3 else (16, 1, 16 * (tiles - 2) - 5)
    ids = list(range(1, len(lens) + 1))
    q, k, v, cu = W.prefill_inputs(layer, lens, seed=tiles + Hkv)
    cfg = S.rope_config(theta=10000.0, rotary_dim=d) if rope else None
    gp = GpuPool(layer, tiles + 2, poison=True)
    gp.ctx.set_partition(32, gp.ctx.device_info()[0] - 32)
    tq, tk, tv = dev_bf16(q), dev_bf16(k), dev_bf16(v)
    wq, wk = dev_bf16(q), dev_bf16(k)
    if rope:
        gp.ctx.rope_qk(PRE, cfg, [i for n in lens for i in range(n)], wq, H, wk, Hkv, d)
    out = torch.empty((cu[-1], H, d), dtype=torch.bfloat16, device=DEV)
    gp.pool.prefill_step(ids, cu, tq, tk, tv, out, H, Hkv, d, d, 1.0 / math.sqrt(d), rope=cfg)
    gp.ctx.phase_sync(PRE)
    np.testing.assert_array_equal(host_bits(tq), host_bits(wq))
    np.testing.assert_array_equal(host_bits(tk), host_bits(wk))
    for i, (r, n) in enumerate(zip(ids, lens)):
        kg = torch.empty((n, Hkv, d), dtype=torch.bfloat16, device=DEV)
        vg = torch.empty_like(kg)
        gp.pool.kv_gather(PRE, r, n, kg, vg)
        gp.ctx.phase_sync(PRE)
        np.testing.assert_array_equal(host_bits(kg), host_bits(wk)[cu[i]:cu[i + 1]])
        np.testing.assert_array_equal(host_bits(vg), v[cu[i]:cu[i + 1]])
    gp.close()
