"""GPU tests of the latent decode step at the sizes where its parts meet: tiles against waves, chunk and page borders, chains of
chunks in one workgroup, both ways of merging them, the new token's row rotated (bf16) or quantised (FP8) into its page."""
import math

import numpy as np
import pytest
import torch

import decode_split as DS
import workloads as W
from oracle import attention as OA
from oracle import fp8 as F8
from oracle import rope as R
from paper_2504_19867_amd import semipd as S
from gpu_util import DEV, GpuPool, assert_parity, dev_bf16, f64, host_bits, host_f64

pytestmark = pytest.mark.gpu
DEC = S.SPD_PHASE_DECODE

CASES = [
    # heads, page tokens, decode CUs, context lengths
    ("tile and wave borders", 16, 64, 256, (1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 192)),
    ("few heads, small pages, merged in the launch", 3, 32, 256, (1000, 33, 4097)),
    ("chains of chunks, merge launch", 16, 64, 32, tuple(40 + 97 * (i % 31) for i in range(70))),
    ("chains of whole requests", 16, 64, 32, tuple(1 + 53 * i % 400 for i in range(150))),
    ("one long request: many chunks", 16, 64, 128, (20001,)),
]


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_latent_decode_appends_and_attends(case, fp8):
    name, H, P, cus, lens = case
    layer = W.LayerShape("mla", H, 1, 192, 128, P, latent_dim=576, latent_v_dim=512)
    gp = GpuPool(layer, sum(-(-n // P) for n in lens) + 8, poison=True, kind=S.SPD_KV_MLA_LATENT_FP8 if fp8 else None)
    total, _, _ = gp.ctx.device_info()
    gp.ctx.set_partition(total, cus)
    rope = None if fp8 else S.rope_config(theta=10000.0, rotary_dim=64, rotary_offset=512)
    o = R.RopeConfig(theta=10000.0, rotary_dim=64)
    q, cs = W.mla_decode_inputs(layer, lens, 5)
    ids = [10 + i for i in range(len(lens))]
    for rid, n, c in zip(ids, lens, cs):
        gp.pool.kv_reserve(rid, max(n - 1, 1))
        if n > 1:
            gp.pool.kv_write(DEC, rid, 0, n - 1, dev_bf16(c[: n - 1]))
    gp.ctx.phase_sync(DEC)
    scale = 1.0 / math.sqrt(192)
    tq, tk = dev_bf16(q), dev_bf16(np.stack([c[-1] for c in cs]))
    out = torch.full((len(lens), H, 512), float("nan"), dtype=torch.bfloat16, device=DEV)
    for _ in range(3):
        gp.pool.decode_step(ids, lens, tq, out, H, scale, k_new=tk, rope=rope)
    again = torch.full_like(out, float("nan"))
    gp.pool.decode_step(ids, lens, tq, again, H, scale, rope=rope)      # with the token in its page: bit for bit
    gp.ctx.phase_sync(DEC)
    assert np.array_equal(host_bits(out), host_bits(again))
    picked = range(len(lens)) if sum(lens) < 30000 else (0, 1, len(lens) // 2, len(lens) - 2, len(lens) - 1)
    for i in picked:
        n, qq = lens[i], f64(q[i])
        if fp8:
            rows = F8.dequantise_latent(*F8.quantise_latent(W.bf16_bits_to_f32(cs[i])))
        else:
            rows = f64(cs[i])
            rows[-1, 512:] = f64(W.to_bf16_bits(R.apply_rope(rows[-1:, None, 512:], [n - 1], o)))[0, 0]
            qq = qq.copy()
            qq[:, 512:] = f64(W.to_bf16_bits(R.apply_rope(qq[None, :, 512:], [n - 1], o)))[0]
        assert_parity(host_f64(out[i:i + 1]), OA.mla_decode_latent(qq, rows, scale, 512)[None], f"{name}: context {n}")
    gp.close()


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("batch", [DS.FULL_CHUNK, (64, 8192, 32, 32)], ids=["every page id", "small pages"])
def test_chunks_as_long_as_the_kernels_page_list(batch, fp8):
    """A small share and much context: chunks of up to as many pages as the workgroup keeps ids of."""
    B, n, P, cus = batch
    H = 16
    layer = W.LayerShape("mla", H, 1, 192, 128, P, latent_dim=576, latent_v_dim=512)
    gp = GpuPool(layer, B * -(-n // P) + 8, poison=True, kind=S.SPD_KV_MLA_LATENT_FP8 if fp8 else None)
    total, _, _ = gp.ctx.device_info()
    gp.ctx.set_partition(total, cus)
    rng = np.random.default_rng(9)
    rows = W.normal_bf16(rng, (n + B, 576))              # request i: rows i .. i + n - 1
    dev = dev_bf16(rows)
    q = W.normal_bf16(rng, (B, H, 576))
    q[..., :512] = W.normal_bf16(rng, (B, H, 512), float(W.MLA_QABS_NOPE_STD))
    ids = [10 + i for i in range(B)]
    for i, rid in enumerate(ids):
        gp.pool.kv_reserve(rid, n - 1)
        gp.pool.kv_write(DEC, rid, 0, n - 1, dev[i:i + n - 1])
    gp.ctx.phase_sync(DEC)
    scale = 1.0 / math.sqrt(192)
    out = torch.full((B, H, 512), float("nan"), dtype=torch.bfloat16, device=DEV)
    tq, new = dev_bf16(q), dev[n - 1:n - 1 + B]
    gp.pool.decode_step(ids, [n] * B, tq, out, H, scale, k_new=new)
    again = torch.full_like(out, float("nan"))
    gp.pool.decode_step(ids, [n] * B, tq, again, H, scale)     # with the token in its page: bit for bit
    gp.ctx.phase_sync(DEC)
    assert np.array_equal(host_bits(out), host_bits(again))
    for i in (0, B // 2, B - 1):
        c = F8.dequantise_latent(*F8.quantise_latent(W.bf16_bits_to_f32(rows[i:i + n]))) if fp8 else f64(rows[i:i + n])
        assert_parity(host_f64(out[i:i + 1]), OA.mla_decode_latent(f64(q[i]), c, scale, 512)[None], f"request {i} of {batch}")
    gp.close()
