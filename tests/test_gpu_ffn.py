"""GPU parity of the gated FFN's first step (C-ABI spd_ffn_gate_up, spd_ffn_pack_gate_up) against the fp64 oracle.

Paper, Evaluation "Implementation based on DistServe": the first two GEMMs of the gated FFN fused into one.
Bar: |got - exact| <= 2^-8 |exact| + 2^-10.  The kernel rounds silu(g) * u once to bf16 (nearest even): half an ulp
is at most 2^-8 of the exact value's magnitude.  Before that, g and u are fp32 sums of `hidden` exact bf16 products:
the expected error is about 2^-24 sqrt(hidden) times partial sums of order one (4e-6 at hidden 4096), the activation
adds a few 2^-24, and the result moves by at most 1.1 |u| dg + |g| du; the absolute term 2^-10 covers all of that with
a wide margin for the generator's scale (|g|, |u| of order one)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import ffn as F
from paper_2504_19867_amd import semipd as S
from ffn_layout import unpack_gate_up
from gpu_util import DEV, dev_bf16, f64, host_bits, host_f64

pytestmark = pytest.mark.gpu
PRE, DEC = S.SPD_PHASE_PREFILL, S.SPD_PHASE_DECODE


def _assert_ffn(got: np.ndarray, want: np.ndarray, what: str):
    assert got.shape == want.shape, (got.shape, want.shape)
    assert np.isfinite(got).all(), what
    bar = 2.0 ** -8 * np.abs(want) + 2.0 ** -10
    err = np.abs(got - want)
    bad = err > bar
    assert not bad.any(), f"{what}: {int(bad.sum())} entries beyond the bar, worst {err[bad].max():.3e}"
    return float(err.max())


def _run(ctx, phase, xb, wgb, wub, poison_out=True):
    T, K = xb.shape
    I = wgb.shape[0]
    x, wg, wu = dev_bf16(xb), dev_bf16(wgb), dev_bf16(wub)
    w_gu = torch.empty((2 * I, K), dtype=torch.bfloat16, device=DEV)
    out = torch.full((max(T, 1), I), float("nan"), dtype=torch.bfloat16, device=DEV)
    ctx.ffn_pack_gate_up(phase, wg, wu, w_gu, K, I)
    ctx.ffn_gate_up(phase, x, w_gu, out, T, K, I)
    ctx.phase_sync(phase)
    return out[:T], w_gu


@pytest.mark.parametrize("T,K,I", [(300, 256, 256), (1, 64, 128), (64, 512, 384), (256, 32, 128), (257, 96, 128), (515, 1024, 512),
                                   (300, 32, 128), (100, 96, 256), (200, 320, 128), (130, 4096, 128)])
def test_gate_up_matches_oracle(T, K, I):
    ctx = S.Context(0)
    xb, wgb, wub = W.ffn_inputs(T, K, I, seed=100 + T)
    out, w_gu = _run(ctx, PRE, xb, wgb, wub)
    # the packed weights are a permutation of 16-byte pieces: read back through the header's index formula
    # (element by element, for the smaller shapes) they are the two matrices bit for bit
    if K * I <= 512 * 384:
        g2, u2 = unpack_gate_up(host_bits(w_gu), K)
        np.testing.assert_array_equal(g2, wgb)
        np.testing.assert_array_equal(u2, wub)
    want = F.gate_up(f64(xb), f64(wgb), f64(wub))
    _assert_ffn(host_f64(out), want, f"ffn T={T} K={K} I={I}")
    ctx.close()


@pytest.mark.parametrize("T", [1, 16, 17, 32, 33, 64, 65, 127, 128, 129])
@pytest.mark.parametrize("K,I,cus", [(32, 128, 0), (288, 128, 0), (512, 256, 0), (544, 384, 0), (800, 3584, 32), (4096, 3584, 32)])
def test_gate_up_streamed_weights(T, K, I, cus):
    """Up to 128 tokens the weights stream through a register ring of 8 slices (eight waves: inter fills the share) or
    16 (four waves): token counts at the edges of the 16-token blocks, slice counts below, at and beyond the rings (1, 9, 16, 17, 25,
    128), an output tensor that is aligned to its entries only, and no row past the batch written."""
    ctx = S.Context(0)
    if cus:
        ctx.set_partition(ctx.device_info()[0] - cus, cus)
    xb, wgb, wub = W.ffn_inputs(T, K, I, seed=1300 + T)
    x, wg, wu = dev_bf16(xb), dev_bf16(wgb), dev_bf16(wub)
    w_gu = torch.empty((2 * I, K), dtype=torch.bfloat16, device=DEV)
    flat = torch.full(((T + 2) * I + 1,), 7.0, dtype=torch.bfloat16, device=DEV)
    out = flat[1:].view(T + 2, I)
    ctx.ffn_pack_gate_up(DEC, wg, wu, w_gu, K, I)
    ctx.ffn_gate_up(DEC, x, w_gu, out, T, K, I)
    ctx.phase_sync(DEC)
    got = host_f64(flat)
    assert got[0] == 7.0 and (got[1 + T * I:] == 7.0).all()
    _assert_ffn(got[1:1 + T * I].reshape(T, I), F.gate_up(f64(xb), f64(wgb), f64(wub)), f"ffn streamed weights T={T} K={K} I={I}")
    ctx.close()


@pytest.mark.parametrize("T", [1, 17, 33, 64, 65])
@pytest.mark.parametrize("K,I,cus,waves", [(288, 3584, 32, 7), (512, 2944, 32, 6), (96, 2432, 32, 5), (544, 2176, 32, 5), (320, 4736, 64, 5)])
def test_gate_up_streamed_weights_by_five_to_seven_waves(T, K, I, cus, waves):
    """Shares that 16-row units fill best with workgroups of five to seven waves (up to 64 tokens): the last workgroup's spare waves
    (2944 / 16 = 184 = 30 x 6 + 4 units, 152 = 30 x 5 + 2, 136 = 27 x 5 + 1, 296 = 59 x 5 + 1) store nothing, and no row past the batch is written."""
    ctx = S.Context(0)
    ctx.set_partition(ctx.device_info()[0] - cus, cus)
    xb, wgb, wub = W.ffn_inputs(T, K, I, seed=2300 + T + I)
    x, wg, wu = dev_bf16(xb), dev_bf16(wgb), dev_bf16(wub)
    w_gu = torch.empty((2 * I, K), dtype=torch.bfloat16, device=DEV)
    out = torch.full((T + 2, I), 7.0, dtype=torch.bfloat16, device=DEV)
    ctx.ffn_pack_gate_up(DEC, wg, wu, w_gu, K, I)
    ctx.ffn_gate_up(DEC, x, w_gu, out, T, K, I)
    ctx.phase_sync(DEC)
    assert (out[T:] == 7.0).all()
    _assert_ffn(host_f64(out[:T]), F.gate_up(f64(xb), f64(wgb), f64(wub)), f"ffn streamed weights, {waves} waves, T={T} K={K} I={I}")
    ctx.close()


@pytest.mark.parametrize("T", [1, 16, 33, 64, 65, 128])
@pytest.mark.parametrize("K", [32, 64, 288, 512, 544, 640, 672, 992, 1024, 1056, 2080])
@pytest.mark.parametrize("I", [896, 1408])
def test_gate_up_streamed_weights_in_two_parts(T, K, I):
    """Shares of more compute units than workgroups of four units would be (32 for 56 and 88 units): workgroups of two or, up to 64
    tokens, three units whose slices two waves share (from hidden 512 on up to 32 tokens, else from 544; below it four units): parts of
    equal and of unequal length at and beyond a ring (8, 9 | 8, 10, 11 | 10, 16 | 15, 16, 17 | 16, 33 | 32 slices), spare waves of the last workgroup (88 = 29 x 3 + 1)."""
    ctx = S.Context(0)
    ctx.set_partition(ctx.device_info()[0] - 32, 32)
    xb, wgb, wub = W.ffn_inputs(T, K, I, seed=3300 + T + I)
    x, wg, wu = dev_bf16(xb), dev_bf16(wgb), dev_bf16(wub)
    w_gu = torch.empty((2 * I, K), dtype=torch.bfloat16, device=DEV)
    out = torch.full((T + 2, I), 7.0, dtype=torch.bfloat16, device=DEV)
    ctx.ffn_pack_gate_up(DEC, wg, wu, w_gu, K, I)
    ctx.ffn_gate_up(DEC, x, w_gu, out, T, K, I)
    ctx.phase_sync(DEC)
    assert (out[T:] == 7.0).all()
    _assert_ffn(host_f64(out[:T]), F.gate_up(f64(xb), f64(wgb), f64(wub)), f"ffn in two parts, T={T} K={K} I={I}")
    ctx.close()


@pytest.mark.parametrize("K", [32, 64, 96, 128, 160, 512])
@pytest.mark.parametrize("T,I,cus", [(1537, 1024, 32), (300, 4224, 32), (257, 1152, 64), (1025, 256, 0)])
def test_gate_up_several_tiles_per_workgroup(T, I, cus, K):
    """Prompt batches on a share of their own: a workgroup takes one to three 256 x 256 tiles (56, 66, 18 of them on 32 or 64 CUs;
    cus = 0: both phases on all of them, one workgroup per tile), the loads three slices ahead of the reads cross from tile to tile
    (1 to 16 slices per tile), token and column counts leave ragged tiles and blocks, the output is aligned to its
    entries only, and nothing is written past the batch."""
    ctx = S.Context(0)
    if cus:
        ctx.set_partition(cus, ctx.device_info()[0] - cus)
    xb, wgb, wub = W.ffn_inputs(T, K, I, seed=1700 + T + K)
    x, wg, wu = dev_bf16(xb), dev_bf16(wgb), dev_bf16(wub)
    w_gu = torch.empty((2 * I, K), dtype=torch.bfloat16, device=DEV)
    flat = torch.full(((T + 2) * I + 1,), 7.0, dtype=torch.bfloat16, device=DEV)
    out = flat[1:].view(T + 2, I)
    ctx.ffn_pack_gate_up(PRE, wg, wu, w_gu, K, I)
    ctx.ffn_gate_up(PRE, x, w_gu, out, T, K, I)
    ctx.phase_sync(PRE)
    got = host_f64(flat)
    assert got[0] == 7.0 and (got[1 + T * I:] == 7.0).all()
    _assert_ffn(got[1:1 + T * I].reshape(T, I), F.gate_up(f64(xb), f64(wgb), f64(wub)), f"ffn tiles T={T} K={K} I={I} cus={cus}")
    ctx.close()


@pytest.mark.parametrize("T", [129, 160, 161, 256])
@pytest.mark.parametrize("K,I", [(96, 2048), (544, 3072)])
def test_gate_up_two_small_tiles_on_some_compute_units(T, K, I):
    """129 to 256 tokens on 32 CUs: 8 and 12 small tiles per XCD, so that one and two compute units more than there are would be needed per
    shader array (the latter up to 160 tokens; above, the large tiles)."""
    ctx = S.Context(0)
    ctx.set_partition(ctx.device_info()[0] - 32, 32)
    xb, wgb, wub = W.ffn_inputs(T, K, I, seed=2900 + T + I)
    x, wg, wu = dev_bf16(xb), dev_bf16(wgb), dev_bf16(wub)
    w_gu = torch.empty((2 * I, K), dtype=torch.bfloat16, device=DEV)
    out = torch.full((T + 2, I), 7.0, dtype=torch.bfloat16, device=DEV)
    ctx.ffn_pack_gate_up(DEC, wg, wu, w_gu, K, I)
    ctx.ffn_gate_up(DEC, x, w_gu, out, T, K, I)
    ctx.phase_sync(DEC)
    assert (out[T:] == 7.0).all()
    _assert_ffn(host_f64(out[:T]), F.gate_up(f64(xb), f64(wgb), f64(wub)), f"ffn small tiles T={T} K={K} I={I}")
    ctx.close()


@pytest.mark.parametrize("T,K,I", [(1, 256, 128), (7, 512, 384), (31, 256, 640), (32, 1024, 128), (33, 256, 128), (48, 768, 256),
                                   (63, 512, 128), (64, 256, 384), (16, 4096, 256), (64, 4096, 128)])
def test_gate_up_batches_of_up_to_64_tokens(T, K, I):
    """At most 64 tokens: the instances for few tokens (which one depends on the phase's share of compute units and on
    inter), ragged token counts, 8 to 128 slices."""
    ctx = S.Context(0)
    xb, wgb, wub = W.ffn_inputs(T, K, I, seed=500 + T)
    for phase in (PRE, DEC):
        out, _ = _run(ctx, phase, xb, wgb, wub)
        _assert_ffn(host_f64(out), F.gate_up(f64(xb), f64(wgb), f64(wub)), f"ffn small batch T={T} K={K} I={I}")
    ctx.close()


@pytest.mark.parametrize("T,K", [(5, 256), (33, 512), (64, 1024)])
def test_gate_up_small_batch_on_a_small_share_takes_the_wide_tile(T, K):
    """inter = 3584 gives 28 workgroups of 256 joint rows: on a 32-CU decode share that is enough for the eight-wave
    instance, which the shapes above never reach on larger shares."""
    ctx = S.Context(0)
    total, _, gran = ctx.device_info()
    ctx.set_partition(total - gran, gran)
    I = 3584
    xb, wgb, wub = W.ffn_inputs(T, K, I, seed=900 + T)
    out, _ = _run(ctx, DEC, xb, wgb, wub)
    assert ctx.get_partition()[1] == gran
    _assert_ffn(host_f64(out), F.gate_up(f64(xb), f64(wgb), f64(wub)), f"ffn small batch, wide tile T={T} K={K}")
    ctx.close()


def test_both_phases_and_partitions_give_the_same_bits():
    ctx = S.Context(0)
    total = ctx.device_info()[0]
    xb, wgb, wub = W.ffn_inputs(700, 256, 640, seed=7)
    ref, _ = _run(ctx, PRE, xb, wgb, wub)
    ref = host_bits(ref)
    ctx.set_partition(total // 4, 3 * total // 4)
    for phase in (PRE, DEC):
        got, _ = _run(ctx, phase, xb, wgb, wub)
        np.testing.assert_array_equal(host_bits(got), ref)
    ctx.close()


def test_rows_past_the_batch_are_not_written_and_zero_tokens_is_a_no_op():
    ctx = S.Context(0)
    T, K, I = 130, 128, 128
    xb, wgb, wub = W.ffn_inputs(T, K, I, seed=9)
    x, wg, wu = dev_bf16(xb), dev_bf16(wgb), dev_bf16(wub)
    w_gu = torch.empty((2 * I, K), dtype=torch.bfloat16, device=DEV)
    out = torch.full((T + 40, I), 7.0, dtype=torch.bfloat16, device=DEV)
    ctx.ffn_pack_gate_up(PRE, wg, wu, w_gu, K, I)
    ctx.ffn_gate_up(PRE, x, w_gu, out, 0, K, I)
    ctx.phase_sync(PRE)
    assert (out == 7.0).all()
    ctx.ffn_gate_up(PRE, x, w_gu, out, T, K, I)
    ctx.phase_sync(PRE)
    assert (out[T:] == 7.0).all()
    _assert_ffn(host_f64(out[:T]), F.gate_up(f64(xb), f64(wgb), f64(wub)), "ffn ragged")
    ctx.close()


def test_large_gate_values_saturate_like_the_definition():
    # silu(z) -> z for large z and -> 0 for very negative z: no NaN from exp overflow
    ctx = S.Context(0)
    T, K, I = 4, 32, 128
    x = np.zeros((T, K), dtype=np.float32)
    x[:, 0] = [100.0, -100.0, 30.0, -30.0]
    wg = np.zeros((I, K), dtype=np.float32)
    wg[:, 0] = 1.0
    wu = np.zeros((I, K), dtype=np.float32)
    wu[:, 0] = 0.5
    xb, wgb, wub = W.to_bf16_bits(x), W.to_bf16_bits(wg), W.to_bf16_bits(wu)
    out, _ = _run(ctx, DEC, xb, wgb, wub)
    _assert_ffn(host_f64(out), F.gate_up(f64(xb), f64(wgb), f64(wub)), "ffn saturation")
    ctx.close()


def test_llama3_8b_shape_sampled():
    """The Llama-3-8B layer shape (hidden 4096, inter 14336) on a prefill batch of 8192 tokens, as the bench times it;
    the oracle checks a sample of token rows, all columns."""
    ctx = S.Context(0)
    T, K, I = 8192, 4096, 14336
    xb, wgb, wub = W.ffn_inputs(T, K, I, seed=2024)
    out, _ = _run(ctx, PRE, xb, wgb, wub)
    rows = np.array([0, 1, 255, 256, 4095, 4096, 5000, 8191])
    want = F.gate_up(f64(xb[rows]), f64(wgb), f64(wub))
    _assert_ffn(host_f64(out[torch.from_numpy(rows).to(DEV)]), want, "ffn llama-3-8b sampled rows")
    ctx.close()


def test_prompt_and_decode_batches_at_the_same_time_on_disjoint_partitions():
    """The paper's setting for this step: a prompt batch on the prefill partition while the decode partition runs
    decode batches; every launch gives the bits it gives alone."""
    ctx = S.Context(0)
    total = ctx.device_info()[0]
    K, I = 512, 1024
    xpb, wgb, wub = W.ffn_inputs(1500, K, I, seed=31)
    xdb, _, _ = W.ffn_inputs(48, K, I, seed=32)
    ref_p, w_gu = _run(ctx, PRE, xpb, wgb, wub)
    ref_p = host_bits(ref_p)
    xd = dev_bf16(xdb)
    od = torch.full((48, I), float("nan"), dtype=torch.bfloat16, device=DEV)
    ctx.ffn_gate_up(DEC, xd, w_gu, od, 48, K, I)
    ctx.phase_sync(DEC)
    ref_d = host_bits(od)
    _assert_ffn(host_f64(od), F.gate_up(f64(xdb), f64(wgb), f64(wub)), "ffn decode batch")
    ctx.set_partition(total // 2, total // 2)
    xp = dev_bf16(xpb)
    outs_p = [torch.full((1500, I), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(3)]
    outs_d = [torch.full((48, I), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(12)]
    for i in range(3):                            # both streams fill up before either drains
        ctx.ffn_gate_up(PRE, xp, w_gu, outs_p[i], 1500, K, I)
        for j in range(4):
            ctx.ffn_gate_up(DEC, xd, w_gu, outs_d[4 * i + j], 48, K, I)
    ctx.phase_sync(PRE)
    ctx.phase_sync(DEC)
    assert ctx.get_partition()[:2] == (total // 2, total // 2)
    for o in outs_p:
        np.testing.assert_array_equal(host_bits(o), ref_p)
    for o in outs_d:
        np.testing.assert_array_equal(host_bits(o), ref_d)
    ctx.close()


def test_random_shapes():
    """Seeded random (tokens, hidden, inter) within the interface's conditions: every tile instance, ragged token
    counts, hidden sizes that are not a multiple of the 64-wide register pipeline's unroll."""
    rng = np.random.default_rng(77)
    ctx = S.Context(0)
    for case in range(12):
        T = int(rng.integers(1, 700))
        K = 32 * int(rng.integers(1, 33))
        I = 128 * int(rng.integers(1, 7))
        xb, wgb, wub = W.ffn_inputs(T, K, I, seed=500 + case)
        out, _ = _run(ctx, (PRE, DEC)[case % 2], xb, wgb, wub)
        _assert_ffn(host_f64(out), F.gate_up(f64(xb), f64(wgb), f64(wub)), f"ffn random case {case}: T={T} K={K} I={I}")
    ctx.close()
