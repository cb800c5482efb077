"""GPU parity of the prefill kernel for 192 / 128 dims (two groups of waves half a tile apart) against the fp64 oracle, through
spd_prefill_step over a latent pool."""
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
SCALE = 1.0 / math.sqrt(192)


def _run(H, lens, cus, make):
    layer = W.LayerShape("gqa", H, H, 192, 128, 16)
    q, k, v, cu = make(layer)
    latent = W.normal_bf16(np.random.default_rng(5), (int(cu[-1]), 576))
    pool_layer = W.LayerShape("mla", H, 1, 192, 128, 64, latent_dim=576, latent_v_dim=512)
    gp = GpuPool(pool_layer, sum(-(-n // 64) for n in lens) + 1)
    if cus:
        gp.ctx.set_partition(cus, gp.ctx.device_info()[0] - cus)
    out = torch.full((q.shape[0] + 1, H, 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    gp.pool.prefill_step([1 + i for i in range(len(lens))], cu, dev_bf16(q), dev_bf16(k), dev_bf16(v), out, H, H, 192, 128, SCALE,
                         latent=dev_bf16(latent))
    gp.ctx.phase_sync(PRE)
    got = host_f64(out)
    assert np.isnan(got[-1]).all()
    gp.close()
    return got[:-1], OA.prefill_attention(f64(q), f64(k), f64(v), cu, SCALE), host_bits(out)


# Chains of one-tile items, item ends on every stage of the rings of three, waves without rows, tiles that only some waves have
# (test_prefill_parts.py asks the host that the whole batch goes to this kernel)
BORDERS = [(3, (1500,) + (1,) * 30 + (64, 65, 63)), (16, (1, 31, 32, 33, 63, 64, 65, 400)), (2, (255, 256, 257, 320, 700)), (1, (1300, 1))]
# batches of the same kind for which prefill_kernel is the faster one
ONE_GROUP = [(3, (385,) + (1,) * 30 + (64, 65, 63)), (2, (384, 383))]


@pytest.mark.parametrize("H,lens", BORDERS + ONE_GROUP)
def test_item_and_tile_borders(H, lens):
    ref = None
    for cus in (32, 0):            # one chain per compute unit; one workgroup per item
        got, want, bits = _run(H, lens, cus, lambda layer: W.prefill_inputs(layer, lens, seed=40 + H))
        assert_parity(got, want, f"prefill 192/128 H={H} cus={cus}")
        if ref is None:
            ref = bits
        np.testing.assert_array_equal(bits, ref)


@pytest.mark.parametrize("rise", [30.0, 400.0, -200.0])
def test_scores_drifting_along_the_keys(rise):
    """The reference of the softmax has to follow the scores, or to stay where the first keys put it."""
    lens = (700, 64, 1, 333)
    got, want, _ = _run(4, lens, 0, lambda layer: W.prefill_inputs_drifting(layer, lens, seed=17, rise=rise, scale=SCALE))
    assert_parity(got, want, f"prefill 192/128 drifting scores rise={rise}")
