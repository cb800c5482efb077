"""The host's dealing of prefill items to chains, parts of items among them, asked through a small program compiled for the CPU: every
tile of every item is visited once whichever way the batch is dealt, and the parts keep the conditions their kernel relies on."""
import os
import random
import shutil
import subprocess

import pytest

from test_gpu_chunked_prefill import AS_ROWS, MANY_PARTS, READ_FROM_PAGES, SHARED_OUT
from test_gpu_prefill_192 import BORDERS, ONE_GROUP

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_19867_amd", "csrc")
# share, persistent, q heads, KV heads, (len, prefix) per request
FEW = [(128, 1, 32, 8, ((893, 4118), (207, 3798), (547, 7358))), (256, 0, 32, 8, ((14, 2805), (7, 2805))), (64, 1, 64, 8, ((1, 8000),)), (128, 1, 32, 8, ((512, 8000),)),
       (256, 0, 32, 8, ((532, 0), (355, 5023), (605, 3058), (867, 2188))), (32, 1, 5, 1, ((300, 4000),)), (96, 1, 8, 8, ((1, 0), (257, 6000)))]
MANY = [(256, 0, 32, 8, ((1500, 0),)), (256, 0, 32, 8, ((1659, 519),)), (128, 1, 64, 8, ((4096, 0),) * 4), (256, 0, 32, 8, ((2048, 0),) * 4), (128, 1, 32, 8, ((30, 0),) * 50), (128, 1, 8, 8, ((128, 0),) * 2)]


def _build(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path / "dump")
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "prefill_parts_dump.cpp"), "-o", exe], check=True)
    return exe


def _deal(tmp_path, batches):
    exe, text = _build(tmp_path), ""
    for whole in (0, 1):
        for share, persistent, H, Hkv, reqs in batches:
            text += " ".join(map(str, (share, persistent, whole, H, Hkv, len(reqs), *(x for r in reqs for x in r)))) + "\n"
    out = iter(subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=300).stdout.split("\n"))
    answers = []
    for _ in range(2 * len(batches)):
        n_chains, n_work, n_merge, looked_at, two_groups = map(int, next(out).split())
        bounds = list(map(int, next(out).split()))
        assert len(bounds) == n_chains + 1 and bounds[0] == 0 and bounds[-1] == n_work and bounds == sorted(bounds)
        work = [tuple(map(int, next(out).split())) for _ in range(n_work)]
        answers.append((bounds, work, [tuple(map(int, next(out).split())) for _ in range(n_merge)], looked_at, two_groups))
    return answers[:len(batches)], answers[len(batches):]


def _end(share, bounds, work):
    """When the last compute unit is done, in tiles: an XCD's workgroups go to its four shader arrays in turn, each to the compute unit
    there that is free first, and none begins ahead of the one before it."""
    per_xcd, end = share // 8, 0
    arrays = 4 if per_xcd % 4 == 0 else 1
    for x in range(8):
        free, begun = [[0] * (per_xcd // arrays) for _ in range(arrays)], 0
        for i, c in enumerate(range(x, len(bounds) - 1, 8)):
            units = free[i % arrays]
            cu = units.index(min(units))
            begun = max(begun, units[cu])
            units[cu] = begun + sum(w[7] - w[6] + 4 + (w[8] >= 0) for w in work[bounds[c]:bounds[c + 1]])
        end = max(end, *(t for units in free for t in units))
    return end


def _check(batch, got, plain):
    share, persistent, H, Hkv, _ = batch
    G = H // Hkv
    hb = next(h for h in (8, 4, 2, 1) if G % h == 0)
    bm = 32 * (8 // hb)
    bounds, work, merge, looked_at, _ = got
    whole = {(w[:6]): w[7] for w in plain[1]}                     # item -> its tiles
    assert len(whole) == len(plain[1]) and all(w[6] == 0 and w[8] == -1 for w in plain[1]) and not plain[2]
    seen = {}
    for w in work:
        seen.setdefault(w[:6], []).append(w[6:])
    assert set(seen) == set(whole)
    parts_of = {}
    for m in merge:
        parts_of[m[:4]] = m[4:]
    n_parts = 0
    for item, ranges in seen.items():
        ranges.sort()
        assert ranges[0][0] == 0 and ranges[-1][1] == whole[item]
        assert all(a[1] == b[0] for a, b in zip(ranges, ranges[1:])) and all(a < b for a, b, _ in ranges)
        if len(ranges) == 1:
            assert ranges[0][2] == -1
            continue
        n_parts += len(ranges)
        first_row_tile = (item[5] + item[2] * bm) // 64
        assert all(a <= first_row_tile for a, _, _ in ranges)     # every row has keys in every part
        assert all(b - a >= 8 for a, b, _ in ranges)
        part0, n = parts_of.pop(item[:4])
        assert n == len(ranges) and [p for _, _, p in ranges] == list(range(part0, part0 + n))
    assert not parts_of                                           # nothing is merged that was not cut
    # the host's search: a handful of tries, each over a part of the items and the chains (a step that nothing overtakes waits for it)
    assert looked_at <= 8 * (len(whole) + share)
    if not persistent:                                            # no workgroup keeps a compute unit that it was not given alone
        assert all(b - a <= 1 for a, b in zip(bounds, bounds[1:]))
    if merge:
        assert not persistent or len(bounds) - 1 == share
        # predicted end of the step: a tenth (of chains at most ten tiles) and the second launch ahead of the whole items
        most = _end(share, bounds, work), _end(share, plain[0], plain[1])
        assert most[0] <= max(most[1] * 9 // 10, most[1] - 10 if persistent else 0) - 6, most
        assert n_parts <= 2 * share + len(merge)
        numbers = sorted(w[8] for w in work if w[8] >= 0)
        assert numbers == list(range(n_parts))
    return len(merge)


def test_items_are_shared_out_where_a_few_long_ones_would_hold_up_the_step(tmp_path):
    got, plain = _deal(tmp_path, FEW + MANY)
    n = [_check(b, g, p) for b, g, p in zip(FEW + MANY, got, plain)]
    assert all(n[:len(FEW)]) and not any(n[len(FEW):]), n


def test_a_step_in_which_no_item_is_cut_has_whole_items(tmp_path):
    """Ranges of keys come with parts: the steps' host side and the kernels take either to mean both."""
    out = subprocess.run([_build(tmp_path), "uncut"], capture_output=True, text=True, check=True, timeout=60).stdout
    assert out.split("\n")[:2] == ["0 0 0 0"] * 2


def test_batches_of_the_gpu_tests_are_shared_out(tmp_path):
    """The tests of parts on the GPU are tests of parts."""
    batches = [(cus or 256, int(cus > 0), H, Hkv, tuple((n, p) for p, n in reqs if p)) for H, Hkv, _, reqs, cus, *_ in [*SHARED_OUT, MANY_PARTS]]
    got, plain = _deal(tmp_path, batches)
    assert all(_check(b, g, p) for b, g, p in zip(batches, got, plain))
    floats = 8 * (128 * 32 + 64)                                     # that a part of 128 dims leaves
    assert sum(w[8] >= 0 for w in got[-1][1]) * floats * 4 > 16 << 20
    one, _ = _deal(tmp_path, [(*batches[-1][:4], batches[-1][4][:1])])
    assert 0 < sum(w[8] >= 0 for w in one[0][1]) * floats * 4 <= 16 << 20


def test_which_chunked_steps_have_dense_rows(tmp_path):
    """Long pieces behind few cached tokens, which the attention over the pages would take longer for; the GPU tests of either way are that."""
    def ask(cases):       # share, q heads, KV heads, dims, RoPE, ((cached, new), ..)
        text = "".join(" ".join(map(str, (*c[:4], int(c[4]), len(c[5]), *(x for p, n in c[5] for x in (n, p))))) + "\n" for c in cases)
        return [int(x) for x in subprocess.run([_build(tmp_path), "rows"], input=text, capture_output=True, text=True, check=True, timeout=60).stdout.split()]

    rows = [(cus or 256, H, Hkv, d, rope, reqs) for H, Hkv, d, _, rope, cus, reqs in AS_ROWS]
    for rope in (False, True):
        rows += [(128, 32, 8, 128, rope, ((100, 2048),) * 4), (128, 32, 8, 128, rope, ((1500, 4096),)), (128, 32, 8, 128, rope, ((1, 128),)),
                 (128, 64, 8, 128, rope, ((6000, 2048),)), (64, 64, 8, 128, rope, ((64, 2048),) * 8), (256, 64, 8, 128, rope, ((64, 512),) * 4),
                 (128, 32, 1, 128, rope, ((100, 4096),)), (256, 32, 8, 128, rope, ((1 << 20, 1 << 20),) * 64)]           # (the last: sums beyond 2^63)
    rows.append((256, 64, 8, 128, True, ((100, 128),) * 12))
    pages = [(256, H, Hkv, d, rope, READ_FROM_PAGES) for H, Hkv, d, rope in ((8, 2, 128, False), (16, 2, 128, True), (4, 1, 64, False), (6, 3, 64, True))]
    for rope in (False, True):
        pages += [(128, 32, 8, 128, rope, ((6000, 1024),) * 4), (128, 32, 8, 128, rope, ((1500, 256),) * 4), (128, 64, 8, 128, rope, ((6000, 256),) * 4),
                  (128, 16, 16, 128, rope, ((1500, 4096),)), (128, 32, 1, 128, rope, ((400, 700),) * 4),
                  (256, 32, 8, 128, rope, ((0, 201), (7680, 1024), (3000, 700), (4000, 600)))]
    pages.append((256, 64, 8, 128, False, ((100, 128),) * 12))
    assert ask(rows) == [1] * len(rows) and ask(pages) == [0] * len(pages)


def _two_groups(lens):
    """Item by item: three times the tiles ahead of the diagonal where both groups of waves have rows, against one per item."""
    gain = 0
    for n in lens:
        for row0 in range(0, n, 256):
            gain += 3 * (row0 // 64) * (min(256, n - row0) > 128) - 1
    return gain > 0


def test_which_kernel_192_dims_take(tmp_path):
    rng = random.Random(4)
    cases = [lens for _, lens in BORDERS + ONE_GROUP]
    assert [_two_groups(lens) for lens in cases] == [True] * len(BORDERS) + [False] * len(ONE_GROUP)
    for _ in range(300):
        top = rng.choice((64, 300, 500, 1500, 8192))
        cases.append(tuple(rng.randint(1, top) for _ in range(rng.randint(1, 60))))
    got, _ = _deal(tmp_path, [(64, 1, 2, 2, tuple((n, 0) for n in lens)) for lens in cases])
    assert [bool(g[4]) for g in got] == [_two_groups(lens) for lens in cases]


def test_random_batches(tmp_path):
    rng = random.Random(3)
    batches = []
    for _ in range(400):
        H, Hkv = rng.choice(((32, 8), (64, 8), (8, 8), (5, 1), (6, 2), (16, 2)))
        top, deep = 2 ** rng.randint(0, 11), 2 ** rng.randint(0, 14)
        reqs = tuple((rng.randint(1, top), rng.choice((0, rng.randint(0, deep)))) for _ in range(rng.randint(1, 12)))
        batches.append((rng.choice((32, 64, 96, 128, 160, 192, 224, 256, 40)), rng.randint(0, 1), H, Hkv, reqs))
    got, plain = _deal(tmp_path, batches)
    assert sum(bool(_check(b, g, p)) for b, g, p in zip(batches, got, plain)) > 20
