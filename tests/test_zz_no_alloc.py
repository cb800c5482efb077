"""The decode step that allocates nothing (spd_decode_step_noalloc), through the C ABI: its output against
spd_decode_step's on the same inputs (same kernels: bit for bit, which is inside the parity bar) and
against the fp64 oracle, on two calls in a row, the second with a smaller batch; the limits are enforced."""
import ctypes as C
import math

import numpy as np
import pytest
import torch

import workloads as W
from oracle import attention as OA
from paper_2504_19867_amd import semipd as S
from test_decode_split import TIGHT
from gpu_util import DEV, GpuPool, assert_parity, dev_bf16, f64, host_bits, host_f64

pytestmark = pytest.mark.gpu
PRE, DEC = S.SPD_PHASE_PREFILL, S.SPD_PHASE_DECODE


def _fill(gp, ctx_lens, seed, first_id):
    L = gp.layer
    q, ks, vs = W.decode_inputs(L, ctx_lens, seed)
    ids = [first_id + i for i in range(len(ctx_lens))]
    for rid, n, kb, vb in zip(ids, ctx_lens, ks, vs):
        gp.pool.kv_reserve(rid, n)
        gp.pool.kv_write(DEC, rid, 0, n, dev_bf16(kb), dev_bf16(vb))
    gp.ctx.phase_sync(DEC)
    return q, ks, vs, ids


def test_noalloc_decode_equals_decode_step_twice_second_call_smaller():
    layer = W.LayerShape("gqa", 32, 8, 128, 128, 16)
    gp = GpuPool(layer, 2048, poison=True)
    gp.ctx.set_partition(128, 128)
    scale = 1.0 / math.sqrt(layer.dim_qk)
    # first call: contexts long enough for several split-K chunks (the partials go through the scratch array);
    # second call: fewer, shorter requests, one of them a single token
    cases = [((3000, 517, 1, 2049, 4096, 16, 33, 1200), 11, 100), ((700, 1, 95), 12, 200)]
    for ctx_lens, seed, first_id in cases:
        q, ks, vs, ids = _fill(gp, ctx_lens, seed, first_id)
        tq = dev_bf16(q)
        out_a = torch.full((len(ids), layer.n_q_heads, layer.dim_v), float("nan"), dtype=torch.bfloat16, device=DEV)
        out_b = torch.full_like(out_a, float("nan"))
        batch_a = gp.pool.make_decode_batch(ids, ctx_lens, tq, out_a, layer.n_q_heads, scale)
        batch_b = gp.pool.make_decode_batch(ids, ctx_lens, tq, out_b, layer.n_q_heads, scale)
        gp.pool.decode_step_batch(batch_a)
        gp.pool.decode_step_noalloc_batch(batch_b)
        gp.ctx.phase_sync(DEC)
        assert np.array_equal(host_bits(out_a), host_bits(out_b)), "noalloc decode differs from spd_decode_step"
        want = np.stack([OA.decode_attention(f64(q[i]), f64(ks[i]), f64(vs[i]), scale) for i in range(len(ids))])
        assert_parity(host_f64(out_b), want, f"noalloc decode, contexts {ctx_lens}")
    gp.close()


def test_noalloc_decode_with_append_and_mla():
    # MLA latent pool, append variant: the new latent row goes to the page in the same call
    layer = W.get_config("c4").layer
    gp = GpuPool(layer, 256)
    gp.ctx.set_partition(128, 128)
    scale = 1.0 / math.sqrt(layer.dim_qk)
    for ctx_lens, seed, first_id in [((1500, 65, 640, 2047), 21, 300), ((64, 3), 22, 400)]:
        q, cs = W.mla_decode_inputs(layer, ctx_lens, seed)
        ids = [first_id + i for i in range(len(ctx_lens))]
        for rid, n, c in zip(ids, ctx_lens, cs):
            if n > 1:
                gp.pool.kv_reserve(rid, n - 1)
                gp.pool.kv_write(DEC, rid, 0, n - 1, dev_bf16(c[: n - 1]))
        gp.ctx.phase_sync(DEC)
        tq = dev_bf16(q)
        new_rows = dev_bf16(np.stack([c[n - 1] for n, c in zip(ctx_lens, cs)]))
        out = torch.full((len(ids), layer.n_q_heads, layer.latent_v_dim), float("nan"), dtype=torch.bfloat16, device=DEV)
        batch = gp.pool.make_decode_batch(ids, ctx_lens, tq, out, layer.n_q_heads, scale, k_new=new_rows)
        gp.pool.decode_step_noalloc_batch(batch)
        gp.ctx.phase_sync(DEC)
        want = np.stack([OA.mla_decode_latent(f64(q[i]), f64(cs[i]), scale, layer.latent_v_dim) for i in range(len(ids))])
        assert_parity(host_f64(out), want, f"noalloc MLA decode with append, contexts {ctx_lens}")
        # the same step again through the allocating entry point, attend only: bit for bit
        out2 = torch.full_like(out, float("nan"))
        gp.pool.decode_step_batch(gp.pool.make_decode_batch(ids, ctx_lens, tq, out2, layer.n_q_heads, scale))
        gp.ctx.phase_sync(DEC)
        assert np.array_equal(host_bits(out), host_bits(out2))
    gp.close()


def test_noalloc_limits_are_enforced_and_change_nothing():
    meta, ws = S.noalloc_limits()
    assert meta == 256 * 1024 and ws == 32 * 1024 * 1024
    layer = W.LayerShape("gqa", 8, 8, 64, 64, 16)
    n_pages = 70000
    gp = GpuPool(layer, n_pages)
    # a block table beyond the metadata limit: one request of 66 000 pages (4 bytes each)
    n = 66000 * 16
    gp.pool.kv_reserve(1, n)
    q = torch.zeros((1, 8, 64), dtype=torch.bfloat16, device=DEV)
    out = torch.zeros((1, 8, 64), dtype=torch.bfloat16, device=DEV)
    before = gp.pool.stats()
    with pytest.raises(S.SpdError) as e:
        gp.pool.decode_step_noalloc_batch(gp.pool.make_decode_batch([1], [n], q, out, 8, 0.125))
    assert e.value.status == S.SPD_ETOOBIG
    assert gp.pool.stats() == before
    gp.close()


def test_noalloc_takes_as_many_requests_as_its_limit_says():
    """16000 requests of one page, nothing appended: 16 bytes each as the limit counts them, a record of 64 each in the ring."""
    layer = W.LayerShape("gqa", 8, 8, 64, 64, 16)
    B = 16000
    gp = GpuPool(layer, B + 8)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    gp.mem.view(torch.bfloat16).normal_(generator=gen)               # any page contents are rows
    lens = [1 + i % 16 for i in range(B)]
    ids = list(range(1, B + 1))
    for i, n in zip(ids, lens):
        gp.pool.kv_reserve(i, n)
    q = torch.randn((B, 8, 64), generator=gen, device=DEV).to(torch.bfloat16)
    out = [torch.full_like(q, float("nan")) for _ in range(2)]
    torch.cuda.synchronize()
    assert 4 * B * 2 + 8 * B <= S.noalloc_limits()[0]
    gp.pool.decode_step_noalloc_batch(gp.pool.make_decode_batch(ids, lens, q, out[0], 8, 0.125))
    gp.pool.decode_step_batch(gp.pool.make_decode_batch(ids, lens, q, out[1], 8, 0.125))
    gp.ctx.phase_sync(DEC)
    assert torch.isfinite(out[0]).all() and np.array_equal(host_bits(out[0]), host_bits(out[1]))
    k, v = (torch.empty((1, 8, 64), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    gp.pool.kv_gather(DEC, 1, 1, k, v)                               # one token: attention is its value
    gp.ctx.phase_sync(DEC)
    assert np.array_equal(host_bits(out[0][0]), host_bits(v[0]))
    gp.close()


def test_noalloc_latent_decode_with_chunks_lengthened_to_fit():
    """A latent batch whose even deal over the workgroups would not fit the workspace (tests/test_decode_split.py): taken, and equal
    to spd_decode_step's within rounding."""
    B, n, P, cus, H = TIGHT[0]
    layer = W.LayerShape("mla", H, 1, 192, 128, P, latent_dim=576, latent_v_dim=512)
    gp = GpuPool(layer, B * -(-n // P) + 8)
    total, _, _ = gp.ctx.device_info()
    gp.ctx.set_partition(total, cus)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(6)
    gp.mem.view(torch.bfloat16).normal_(generator=gen)
    ids = list(range(1, B + 1))
    for i in ids:
        gp.pool.kv_reserve(i, n)
    q = torch.randn((B, H, 576), generator=gen, device=DEV).mul_(0.2).to(torch.bfloat16)
    out = [torch.full((B, H, 512), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    torch.cuda.synchronize()
    scale = 1.0 / math.sqrt(192)
    gp.pool.decode_step_noalloc_batch(gp.pool.make_decode_batch(ids, [n] * B, q, out[0], H, scale))
    gp.pool.decode_step_batch(gp.pool.make_decode_batch(ids, [n] * B, q, out[1], H, scale))
    gp.ctx.phase_sync(DEC)
    rows = torch.empty((n, 576), dtype=torch.bfloat16, device=DEV)
    for i in (0, B // 2, B - 1):
        gp.pool.kv_gather(DEC, ids[i], n, rows)
        gp.ctx.phase_sync(DEC)
        want = OA.mla_decode_latent(host_f64(q[i]), host_f64(rows), scale, 512)[None]
        for o in out:
            assert_parity(host_f64(o[i:i + 1]), want, f"request {i}")
    # two bf16 roundings of sums whose bf16 weights differ by their rounding: 2^-8 of the largest output, which is below 1
    assert (out[0].float() - out[1].float()).abs().max() < 2 ** -7
    gp.close()


@pytest.mark.parametrize("lens", [(700, 33, 1), tuple(300 + 37 * (i % 29) for i in range(90))], ids=["few", "many"])
def test_noalloc_decode_in_a_graph(lens):
    """Captured on the phase's stream, then replayed with other steps, other batches and other RoPE configurations in between: every
    replay gives what the eager call gives for the query that is there at the time."""
    hip = S.lib                                          # (the runtime that the library is linked to)
    layer = W.LayerShape("gqa", 8, 8, 128, 128, 16)
    gp = GpuPool(layer, sum(-(-n // 16) for n in lens) + 8)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(8)
    gp.mem.view(torch.bfloat16).normal_(generator=gen)   # any page contents are rows
    ids = list(range(1, len(lens) + 1))
    for i, n in zip(ids, lens):
        gp.pool.kv_reserve(i, n)
    cfg, other = S.rope_config(theta=500000.0, factor=8.0), S.rope_config(theta=10000.0)
    q = torch.empty((len(lens), 8, 128), dtype=torch.bfloat16, device=DEV).normal_(generator=gen)
    out, eager, scrap = (torch.full_like(q, float("nan")) for _ in range(3))
    batch = gp.pool.make_decode_batch(ids, lens, q, out, 8, 0.09, rope=cfg)
    torch.cuda.synchronize()
    stream = C.c_void_p(gp.ctx.phase_stream(DEC))
    gp.pool.decode_step(ids, lens, q, scrap, 8, 0.09, rope=other)
    gp.ctx.phase_sync(DEC)
    graph, run = C.c_void_p(), C.c_void_p()
    assert hip.hipStreamBeginCapture(stream, 1) == 0     # thread local
    gp.pool.decode_step_noalloc_batch(batch)
    assert hip.hipStreamEndCapture(stream, C.byref(graph)) == 0
    assert hip.hipGraphInstantiate(C.byref(run), graph, None, None, C.c_uint64(0)) == 0
    for round in range(4):
        gp.pool.decode_step(ids, lens, q, eager, 8, 0.09, rope=cfg)
        for i in range(12):                              # more than there are staging slots
            gp.pool.decode_step(ids[:1 + i % 3], lens[:1 + i % 3], q, scrap, 8, 0.05, rope=other)
        if round % 2:
            gp.ctx.phase_sync(DEC)
        assert hip.hipGraphLaunch(run, stream) == 0
        gp.pool.decode_step(ids, lens, q, scrap, 8, 0.09, rope=other)
        gp.ctx.phase_sync(DEC)
        assert torch.isfinite(eager).all() and np.array_equal(host_bits(out), host_bits(eager)), f"replay {round}"
        q.normal_(generator=gen)
        out.fill_(float("nan"))
        torch.cuda.synchronize()
    gp.ctx.phase_sync(DEC)
    assert hip.hipGraphExecDestroy(run) == 0 and hip.hipGraphDestroy(graph) == 0
    for i in ids:
        gp.pool.kv_free(i)
    gp.close()
