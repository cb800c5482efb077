"""GPU parity of chunked prefill: a prompt processed piece by piece, each piece attending to the
pages written by the pieces before it, against the fp64 oracle (chunk_attention, which is pinned
to the rows of whole-prompt causal attention)."""
import math

import numpy as np
import pytest
import torch

import workloads as W
from oracle import attention as OA
from oracle.allocator import BlockAllocator
from paper_2504_19867_amd import semipd as S
from gpu_util import DEV, GpuPool, assert_parity, dev_bf16, f64, host_bits, host_f64

pytestmark = pytest.mark.gpu
PRE, DEC = S.SPD_PHASE_PREFILL, S.SPD_PHASE_DECODE


def run_chunks(gp, q, k, v, cu, cuts_per_req, ids, scale):
    """Feed each request's rows in the pieces given by its cut list; all requests advance together,
    a request that has run out of pieces simply drops out of the later steps.  Returns the outputs
    [T, H, dv] assembled from the steps."""
    L = gp.layer
    out_all = torch.zeros((q.shape[0], L.n_q_heads, L.dim_v), dtype=torch.bfloat16, device=DEV)
    n_steps = max(len(c) - 1 for c in cuts_per_req)
    for s in range(n_steps):
        rows, step_ids, pre, lens = [], [], [], []
        for r, cuts in enumerate(cuts_per_req):
            if s + 1 < len(cuts):
                a, b = cu[r] + cuts[s], cu[r] + cuts[s + 1]
                rows.append(np.arange(a, b))
                step_ids.append(ids[r])
                pre.append(cuts[s])
                lens.append(b - a)
        idx = np.concatenate(rows)
        step_cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        out = torch.empty((len(idx), L.n_q_heads, L.dim_v), dtype=torch.bfloat16, device=DEV)
        gp.pool.prefill_step(step_ids, step_cu, dev_bf16(q[idx]), dev_bf16(k[idx]), dev_bf16(v[idx]), out, L.n_q_heads,
                             L.n_kv_heads, L.dim_qk, L.dim_v, scale, prefix_lens=pre)
        gp.ctx.phase_sync(PRE)
        out_all[torch.from_numpy(idx).to(DEV)] = out
    return out_all


@pytest.mark.parametrize("H,Hkv,d", [(8, 2, 128), (16, 2, 128), (3, 3, 64)])
def test_chunked_prefill_matches_oracle_and_pages(H, Hkv, d):
    layer = W.LayerShape("gqa", H, Hkv, d, d, 16)
    lens = (300, 77, 513, 16)
    # cut points inside each request: pieces that end mid-tile, mid-page, of one token, and one request in a single piece
    cuts = [[0, 64, 65, 130, 300], [0, 5, 77], [0, 100, 101, 357, 513], [0, 16]]
    gp = GpuPool(layer, 128, poison=True)
    ora = BlockAllocator(128, 16)
    for op, r, n in W.scramble_ops(60, 16, seed=7):
        (gp.pool.kv_reserve(r, n), ora.reserve(r, n)) if op == "reserve" else (gp.pool.kv_free(r), ora.free(r))
    q, k, v, cu = W.prefill_inputs(layer, lens, seed=51 + H)
    scale = 1.0 / math.sqrt(d)
    ids = [11, 12, 13, 14]
    out = run_chunks(gp, q, k, v, cu, cuts, ids, scale)
    got = host_f64(out)
    for r in range(len(lens)):
        for a, b in zip(cuts[r][:-1], cuts[r][1:]):
            want = OA.chunk_attention(f64(q[cu[r] + a:cu[r] + b]), f64(k[cu[r]:cu[r] + b]), f64(v[cu[r]:cu[r] + b]), scale)
            assert_parity(got[cu[r] + a:cu[r] + b], want, f"request {r} piece [{a},{b})")
    # the pages hold the whole prompt, bit for bit, and the tables grew like the oracle's
    for step in range(max(len(c) - 1 for c in cuts)):          # same order as the steps took them
        for r, rid in enumerate(ids):
            if step + 1 < len(cuts[r]):
                ora.reserve(rid, cuts[r][step + 1])
    for r, rid in enumerate(ids):
        assert gp.pool.kv_block_table(rid) == ora.block_table(rid)
        kb = torch.empty((lens[r], Hkv, d), dtype=torch.bfloat16, device=DEV)
        vb = torch.empty((lens[r], Hkv, d), dtype=torch.bfloat16, device=DEV)
        gp.pool.kv_gather(PRE, rid, lens[r], kb, vb)
        gp.ctx.phase_sync(PRE)
        np.testing.assert_array_equal(host_bits(kb), k[cu[r]:cu[r + 1]])
        np.testing.assert_array_equal(host_bits(vb), v[cu[r]:cu[r + 1]])
    # and a decode step over them sees the same context
    qd, _, _ = W.decode_inputs(layer, (1,) * len(lens), seed=99)
    od = torch.empty((len(lens), H, d), dtype=torch.bfloat16, device=DEV)
    gp.ctx.phase_wait_for(DEC, PRE)
    gp.pool.decode_step(ids, lens, dev_bf16(qd), od, H, scale)
    gp.ctx.phase_sync(DEC)
    want_d = np.stack([OA.decode_attention(f64(qd[r]), f64(k[cu[r]:cu[r + 1]]), f64(v[cu[r]:cu[r + 1]]), scale) for r in range(len(lens))])
    assert_parity(host_f64(od), want_d, "decode after chunked prefill")
    gp.close()


def test_chunked_prefill_long_prefix_and_argument_checks():
    layer = W.LayerShape("gqa", 8, 2, 128, 128, 16)
    gp = GpuPool(layer, 400, poison=True)
    n = 4096 + 37
    q, k, v, cu = W.prefill_inputs(layer, (n,), seed=77)
    scale = 1.0 / math.sqrt(128)
    out = run_chunks(gp, q, k, v, cu, [[0, 4000, n]], [5], scale)
    a = 4000
    want = OA.chunk_attention(f64(q[a:n]), f64(k[:n]), f64(v[:n]), scale)
    assert_parity(host_f64(out)[a:n], want, "piece of 133 rows after a prefix of 4000")
    # a prefix that is not there
    one = dev_bf16(q[:8])
    kk, vv = dev_bf16(k[:8]), dev_bf16(v[:8])
    o = torch.empty((8, 8, 128), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(S.SpdError) as e:
        gp.pool.prefill_step([99], [0, 8], one, kk, vv, o, 8, 2, 128, 128, scale, prefix_lens=[32])
    assert e.value.status == S.SPD_ENOENT
    gp.pool.kv_reserve(98, 16)
    with pytest.raises(S.SpdError) as e:
        gp.pool.prefill_step([98], [0, 8], one, kk, vv, o, 8, 2, 128, 128, scale, prefix_lens=[32])
    assert e.value.status == S.SPD_EINVAL
    with pytest.raises(S.SpdError):
        gp.pool.prefill_step([98], [0, 8], one, kk, vv, o, 8, 2, 128, 128, scale, prefix_lens=[-1])
    # exhaustion changes nothing: 400 pages cannot take another 4096-token piece
    free_before = gp.pool.kv_free_list()
    big = dev_bf16(q[:4096])
    ob = torch.empty((4096, 8, 128), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(S.PoolExhausted):
        gp.pool.prefill_step([5], [0, 4096], big, dev_bf16(k[:4096]), dev_bf16(v[:4096]), ob, 8, 2, 128, 128, scale, prefix_lens=[n])
    assert gp.pool.kv_free_list() == free_before
    gp.close()


def test_workspace_grows_between_steps_in_flight():
    """Two chunked steps issued back to back without a wait between them, the second with a context that
    no longer fits the gather workspace of the first (16 MiB to start with): the first step still reads the
    old workspace when the second takes a new one, and both come out right."""
    layer = W.LayerShape("gqa", 8, 2, 64, 64, 16)              # 512 bytes of K and V per cached row
    small, big = 600, 33000                                     # 0.3 MiB, then 16.9 MiB of gathered context
    gp = GpuPool(layer, (small + big) // 16 + 8, poison=True)
    scale = 1.0 / math.sqrt(64)
    qs, ks, vs, _ = W.prefill_inputs(layer, (small,), seed=311)
    qb, kb, vb, _ = W.prefill_inputs(layer, (big,), seed=312)
    cut_s, cut_b = small - 40, big - 24
    # the prefixes, each in one un-chunked step (no workspace), then drained
    for rid, (q, k, v, cut) in ((1, (qs, ks, vs, cut_s)), (2, (qb, kb, vb, cut_b))):
        o = torch.empty((cut, 8, 64), dtype=torch.bfloat16, device=DEV)
        gp.pool.prefill_step([rid], [0, cut], dev_bf16(q[:cut]), dev_bf16(k[:cut]), dev_bf16(v[:cut]), o, 8, 2, 64, 64, scale)
    gp.ctx.phase_sync(PRE)
    out_s = torch.empty((small - cut_s, 8, 64), dtype=torch.bfloat16, device=DEV)
    out_b = torch.empty((big - cut_b, 8, 64), dtype=torch.bfloat16, device=DEV)
    args_s = [dev_bf16(x[cut_s:]) for x in (qs, ks, vs)]
    args_b = [dev_bf16(x[cut_b:]) for x in (qb, kb, vb)]
    gp.pool.prefill_step([1], [0, small - cut_s], *args_s, out_s, 8, 2, 64, 64, scale, prefix_lens=[cut_s])
    gp.pool.prefill_step([2], [0, big - cut_b], *args_b, out_b, 8, 2, 64, 64, scale, prefix_lens=[cut_b])
    gp.ctx.phase_sync(PRE)
    want_s = OA.chunk_attention(f64(qs[cut_s:]), f64(ks), f64(vs), scale)
    want_b = OA.chunk_attention(f64(qb[cut_b:]), f64(kb), f64(vb), scale)
    assert_parity(host_f64(out_s), want_s, "step that read the workspace before it grew")
    assert_parity(host_f64(out_b), want_b, "step that made it grow")
    gp.close()


# heads, dims, (prefix, piece) per request, CUs of a share of its own (0: all of them, with the other phase), drift of the scores in nats
# (test_prefill_parts.py asks the host's dealing that items of every one of them are cut)
SHARED_OUT = [
    (8, 2, 128, ((2805, 14), (1500, 7)), 0, 0.0),                  # parts of one length, rows past the piece
    (16, 2, 128, ((3000, 1),), 64, 0.0),                           # one token
    (8, 2, 128, ((2048, 129), (2111, 64), (0, 40)), 32, 0.0),      # a prefix that ends on a tile, pieces of several items
    (3, 3, 64, ((1984, 300), (100, 33)), 32, 0.0),                 # 64 dims, 256 rows per item, waves whose rows begin behind a part's tiles
    (5, 1, 128, ((2500, 70),), 96, 0.0),
    (8, 2, 128, ((2000, 50),), 0, 300.0),                          # references far apart
    (8, 2, 128, ((2000, 50),), 0, -300.0),
]
MANY_PARTS = (8, 8, 128, ((4000, 1),) * 4, 0)                      # more parts than the buffer of their sums holds at first (16 MiB)


@pytest.mark.parametrize("H,Hkv,d,reqs,cus,rise", SHARED_OUT)
def test_items_shared_out_by_keys(H, Hkv, d, reqs, cus, rise):
    """Few items behind long prefixes: their keys go to several workgroups, whose sums a second launch adds up."""
    layer = W.LayerShape("gqa", H, Hkv, d, d, 16)
    lens = tuple(p + n for p, n in reqs)
    scale = 1.0 / math.sqrt(d)
    q, k, v, cu = W.prefill_inputs_drifting(layer, lens, seed=7 + H, rise=rise, scale=scale) if rise else W.prefill_inputs(layer, lens, seed=7 + H)
    gp = GpuPool(layer, sum(-(-n // 16) for n in lens) + 4, poison=True)
    if cus:
        gp.ctx.set_partition(cus, gp.ctx.device_info()[0] - cus)
    cuts = [[0, p, p + n] if p else [0, n] for p, n in reqs]
    outs = []
    for _ in range(2):
        out = run_chunks(gp, q, k, v, cu, cuts, [1 + i for i in range(len(reqs))], scale)
        outs.append(host_bits(out))
        for i in range(len(reqs)):
            gp.pool.kv_free(1 + i)
    np.testing.assert_array_equal(outs[0], outs[1])
    got = host_f64(out)
    for r, (p, n) in enumerate(reqs):
        want = OA.chunk_attention(f64(q[cu[r] + p:cu[r + 1]]), f64(k[cu[r]:cu[r + 1]]), f64(v[cu[r]:cu[r + 1]]), scale)
        assert_parity(got[cu[r] + p:cu[r + 1]], want, f"request {r}: {n} tokens behind {p}")
    gp.close()


def test_buffer_of_the_parts_sums_grows_between_steps_in_flight():
    """Two steps with shared-out items issued back to back, the second with more parts than the buffer holds that the first one's sums
    went to: the first still writes and reads it when the second takes a new one."""
    H, Hkv, d, reqs, _ = MANY_PARTS
    layer = W.LayerShape("gqa", H, Hkv, d, d, 16)
    scale = 1.0 / math.sqrt(d)
    lens = tuple(p + n for p, n in reqs)
    q, k, v, cu = W.prefill_inputs(layer, lens, seed=61)
    gp = GpuPool(layer, sum(-(-n // 16) for n in lens) + 4, poison=True)
    for r, (p, _) in enumerate(reqs):
        gp.pool.kv_reserve(1 + r, p)
        gp.pool.kv_write(PRE, 1 + r, 0, p, dev_bf16(k[cu[r]:cu[r] + p]), dev_bf16(v[cu[r]:cu[r] + p]))
    gp.ctx.phase_sync(PRE)
    outs = []
    for first, last in ((0, 1), (0, len(reqs)), (0, 1)):              # one request, all of them, one again (its pieces written anew)
        rows = np.concatenate([np.arange(cu[r] + reqs[r][0], cu[r + 1]) for r in range(first, last)])
        outs.append(([dev_bf16(x[rows]) for x in (q, k, v)], torch.empty((len(rows), H, d), dtype=torch.bfloat16, device=DEV), last))
    torch.cuda.synchronize()
    for step, out, last in outs:
        gp.pool.prefill_step([1 + r for r in range(last)], list(range(last + 1)), *step, out, H, Hkv, d, d, scale, prefix_lens=[p for p, _ in reqs[:last]])
    gp.ctx.phase_sync(PRE)
    want = np.concatenate([OA.chunk_attention(f64(q[cu[r] + p:cu[r + 1]]), f64(k[cu[r]:cu[r + 1]]), f64(v[cu[r]:cu[r + 1]]), scale) for r, (p, _) in enumerate(reqs)])
    for i, (_, out, last) in enumerate(outs):
        assert_parity(host_f64(out), want[:last], f"step {i}")
    gp.close()


@pytest.mark.parametrize("H,Hkv,d,bits", [(16, 2, 128, 0xFF80), (16, 2, 128, 0xFF7F), (8, 8, 64, 0xFF80)])     # -inf, the lowest finite value
def test_items_shared_out_whose_parts_see_only_masked_keys(H, Hkv, d, bits):
    """Keys that no query can choose (scores of -inf, or so low that fp32 takes them there) from the second tile of the prefix to its
    end: whole parts of the item hold nothing else, and they weigh nothing."""
    prefix, n = 3000, 5
    layer = W.LayerShape("gqa", H, Hkv, d, d, 16)
    scale = 1.0 / math.sqrt(d)
    q, k, v, cu = W.prefill_inputs(layer, (prefix + n,), seed=5)
    q, k = q.copy(), k.copy()
    q[prefix:, :, 0] = 0x4080                                        # 4.0
    k[64:prefix, :, 0] = bits
    gp = GpuPool(layer, -(-(prefix + n) // 16) + 4, poison=True)
    gp.ctx.set_partition(64, gp.ctx.device_info()[0] - 64)
    # the prefix is written as pages, not computed: its own rows see only masked keys
    gp.pool.kv_reserve(1, prefix)
    gp.pool.kv_write(PRE, 1, 0, prefix, dev_bf16(k[:prefix]), dev_bf16(v[:prefix]))
    out = torch.empty((n, H, d), dtype=torch.bfloat16, device=DEV)
    gp.pool.prefill_step([1], [0, n], dev_bf16(q[prefix:]), dev_bf16(k[prefix:]), dev_bf16(v[prefix:]), out, H, Hkv, d, d, scale, prefix_lens=[prefix])
    gp.ctx.phase_sync(PRE)
    want = OA.chunk_attention(f64(q[prefix:]), f64(k), f64(v), scale)
    assert_parity(host_f64(out), want, f"{n} tokens behind {prefix}, keys 64 .. {prefix - 1} masked")
    gp.close()


@pytest.mark.parametrize("pre,dec", [(256, 256), (192, 192)])
def test_decode_steps_beside_items_shared_out_on_the_same_compute_units(pre, dec):
    """Parts are workgroups of their own where the phases' masks overlap: both phases' steps, issued in turn, end and are right."""
    H, Hkv, d, reqs, n_dec, n_ctx = 8, 2, 128, ((2805, 70), (1500, 7)), 6, 300
    layer = W.LayerShape("gqa", H, Hkv, d, d, 16)
    scale = 1.0 / math.sqrt(d)
    lens = tuple(p + n for p, n in reqs)
    q, k, v, cu = W.prefill_inputs(layer, lens, seed=23)
    qd, ks, vs = W.decode_inputs(layer, (n_ctx,) * n_dec, 24)
    gp = GpuPool(layer, sum(-(-n // 16) for n in lens) + n_dec * -(-n_ctx // 16) + 4, poison=True)
    gp.ctx.set_partition(pre, dec)
    for i, (kb, vb) in enumerate(zip(ks, vs)):
        gp.pool.kv_reserve(50 + i, n_ctx)
        gp.pool.kv_write(DEC, 50 + i, 0, n_ctx, dev_bf16(kb), dev_bf16(vb))
    for r, (p, _) in enumerate(reqs):
        gp.pool.kv_reserve(1 + r, p)
        gp.pool.kv_write(PRE, 1 + r, 0, p, dev_bf16(k[cu[r]:cu[r] + p]), dev_bf16(v[cu[r]:cu[r] + p]))
    gp.ctx.phase_sync(PRE)
    gp.ctx.phase_sync(DEC)
    rows = np.concatenate([np.arange(cu[r] + p, cu[r + 1]) for r, (p, _) in enumerate(reqs)])
    step = [dev_bf16(x[rows]) for x in (q, k, v)]
    cu_step = [0, reqs[0][1], reqs[0][1] + reqs[1][1]]
    out_p = torch.empty((len(rows), H, d), dtype=torch.bfloat16, device=DEV)
    tqd, out_d = dev_bf16(qd), torch.empty((n_dec, H, d), dtype=torch.bfloat16, device=DEV)
    torch.cuda.synchronize()
    for _ in range(4):
        gp.pool.prefill_step([1, 2], cu_step, *step, out_p, H, Hkv, d, d, scale, prefix_lens=[p for p, _ in reqs])
        gp.pool.decode_step([50 + i for i in range(n_dec)], [n_ctx] * n_dec, tqd, out_d, H, scale)
    gp.ctx.phase_sync(PRE)
    gp.ctx.phase_sync(DEC)
    got = host_f64(out_p)
    for r, (p, n) in enumerate(reqs):
        want = OA.chunk_attention(f64(q[cu[r] + p:cu[r + 1]]), f64(k[cu[r]:cu[r + 1]]), f64(v[cu[r]:cu[r + 1]]), scale)
        assert_parity(got[cu_step[r]:cu_step[r + 1]], want, f"request {r}")
    want_d = np.stack([OA.decode_attention(f64(qd[i]), f64(ks[i]), f64(vs[i]), scale) for i in range(n_dec)])
    assert_parity(host_f64(out_d), want_d, "decode")
    gp.close()


# (cached tokens, new ones) per request
READ_FROM_PAGES = ((1023, 1), (1024, 33), (1025, 64), (2050, 13), (0, 70), (15, 2), (64, 129))
FEW_CACHED = ((1, 300), (17, 129), (0, 70), (100, 64), (15, 2), (64, 65), (3, 13))
# q heads, KV heads, dims, page tokens, RoPE, compute units (0: all), requests
AS_ROWS = [(8, 2, 128, 16, False, 0, FEW_CACHED), (16, 2, 128, 64, True, 0, FEW_CACHED), (6, 3, 64, 48, True, 0, FEW_CACHED), (4, 4, 64, 32, False, 0, FEW_CACHED),
           (16, 16, 128, 16, True, 0, FEW_CACHED[:3]), (16, 1, 128, 32, True, 32, ((40, 2300), (17, 70)))]


def _check_pieces(H, Hkv, d, page, rope, reqs, cus=0):
    """One step of the requests' pieces, pages in no order and NaN behind the tokens."""
    layer = W.LayerShape("gqa", H, Hkv, d, d, page)
    scale = 1.0 / math.sqrt(d)
    lens = tuple(p + n for p, n in reqs)
    q, k, v, cu = W.prefill_inputs(layer, lens, seed=29 + H)
    gp = GpuPool(layer, sum(-(-n // page) for n in lens) + 70, poison=True)
    for op, r, n in W.scramble_ops(60, page, seed=7):
        (gp.pool.kv_reserve if op == "reserve" else lambda r, _: gp.pool.kv_free(r))(r, n)
    if cus:
        gp.ctx.set_partition(cus, 256 - cus)
    for r, (p, _) in enumerate(reqs):
        if p:
            gp.pool.kv_reserve(1 + r, p)
            gp.pool.kv_write(PRE, 1 + r, 0, p, dev_bf16(k[cu[r]:cu[r] + p]), dev_bf16(v[cu[r]:cu[r] + p]))
    rows = np.concatenate([np.arange(cu[r] + p, cu[r + 1]) for r, (p, _) in enumerate(reqs)])
    cu_step = np.concatenate([[0], np.cumsum([n for _, n in reqs])]).astype(np.int64)
    tq, tk, tv = [dev_bf16(x[rows]) for x in (q, k, v)]
    out = torch.empty((len(rows), H, d), dtype=torch.bfloat16, device=DEV)
    cfg = S.rope_config(theta=10000.0, rotary_dim=d) if rope else None
    gp.pool.prefill_step([1 + r for r in range(len(reqs))], cu_step, tq, tk, tv, out, H, Hkv, d, d, scale, prefix_lens=[p for p, _ in reqs], rope=cfg)
    gp.ctx.phase_sync(PRE)
    got, q_used, k_used = host_f64(out), host_f64(tq), host_f64(tk)      # (rotated in place with rope)
    for r, (p, n) in enumerate(reqs):
        a, b = cu_step[r], cu_step[r + 1]
        keys = np.concatenate([f64(k[cu[r]:cu[r] + p]), k_used[a:b]])
        assert_parity(got[a:b], OA.chunk_attention(q_used[a:b], keys, f64(v[cu[r]:cu[r + 1]]), scale), f"request {r}: {n} tokens behind {p}")
    gp.close()


@pytest.mark.parametrize("H,Hkv,d,page,rope", [(8, 2, 128, 16, False), (16, 2, 128, 64, True), (4, 1, 64, 32, False), (6, 3, 64, 48, True)])
def test_pieces_read_from_scattered_pages(H, Hkv, d, page, rope):
    """Keys and values come out of the pages: pages of one and of several units of 16 tokens in no order, prefixes around the 1024 tokens whose units
    a workgroup has at hand, ends in every part of a unit, and NaN behind them."""
    _check_pieces(H, Hkv, d, page, rope, READ_FROM_PAGES)


@pytest.mark.parametrize("H,Hkv,d,page,rope,cus,reqs", AS_ROWS)
def test_pieces_brought_together_as_rows(H, Hkv, d, page, rope, cus, reqs):
    """The same where the step brings keys and values together as dense rows: prefixes and pieces that end in every part of a unit, and one KV
    head, whose rows a launch of their own gathers (test_prefill_parts.py has that these are such steps)."""
    _check_pieces(H, Hkv, d, page, rope, reqs, cus)
