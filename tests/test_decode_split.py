"""Host logic, no GPU: every tile of a decode batch belongs to one chunk, chains of chunks are walks through all of them, and
no chunk of the latent decode touches more pages than its kernel has room for."""
import heapq
import random

import pytest

import decode_split as DS

TILE = 16
KERNEL_THREADS = 256                # of a latent workgroup, which fetches a record one word per thread

# requests, context, page tokens, decode CUs: batches whose even share of a workgroup is longer than the kernel's page list
LONG = [(64, 8192, 32, 32), (16, 32768, 32, 32), (64, 16384, 64, 32), (128, 8192, 32, 64), (128, 16384, 64, 64), (130, 16384, 64, 64),
        (128, 16384, 32, 128), (256, 8192, 32, 128), (1, 1000000, 32, 32), (8, 300000, 96, 32), (2, 4000000, 1024, 32),
        (40, 1000000, 1024, 256), DS.FULL_CHUNK]


def _random_batches():
    rng = random.Random(3)
    for _ in range(150):
        B = rng.choice((1, 2, 3, 7, 20, 64, 200))
        top = rng.choice((16, 200, 4000, 30000))
        lens = [rng.randint(1, top) if rng.random() < 0.9 else 8 * top for _ in range(B)]
        yield lens, rng.choice((32, 64, 96, 1024)), rng.choice((32, 64, 96, 128, 256)), rng.choice((0, 0, 0, 1, 5, 40))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return DS.build(tmp_path_factory.mktemp("split"))


def _pages(unit0, n, per_page):
    return (unit0 + n - 1) // per_page - unit0 // per_page + 1


def _check_cover(items, lens):
    by_req = {}
    for req, chunk, u0, n, _ in items:
        by_req.setdefault(req, []).append((chunk, u0, n))
    assert sorted(by_req) == list(range(len(lens)))
    for r, chunks in by_req.items():
        at = 0
        for i, (chunk, u0, n) in enumerate(sorted(chunks)):
            assert chunk == i and u0 == at and n > 0
            at += n
        assert at == -(-lens[r] // TILE)


@pytest.mark.parametrize("kind", ["latent", "latent_fp8"])
def test_latent_chunks_fit_the_kernel(exe, kind):
    batches = [(kind, P, cus, 1, 16, 1, 0, [n] * B) for B, n, P, cus in LONG]
    batches += [(kind, P, cus, 1, 16, 1, o, lens) for lens, P, cus, o in _random_batches()]
    (room, words, *_), answers = DS.split(exe, batches)
    assert room + words <= KERNEL_THREADS
    longest = 0
    for (_, P, cus, _, _, _, override, lens), s in zip(batches, answers):
        per_page = P // TILE
        most = max(_pages(u0, n, per_page) for _, _, u0, n, _ in s.items)
        longest = max(longest, most)
        assert most <= room, (P, cus, len(lens), most)
        # the record as the host lays it out, rounded up to 64 bytes
        assert s.record_bytes >= len(s.items) * 4 * (words + most)
        assert s.record_bytes <= len(s.items) * 4 * KERNEL_THREADS + 4 * len(lens) + 16
        _check_cover(s.items, lens)
        assert s.max_chunks == max(i[1] for i in s.items) + 1 and s.chunk_units == max(i[3] for i in s.items)
        assert override or s.n_wgs <= 2 * cus
        # the chains that workgroups 0 .. n_wgs - 1 walk pass through every item once
        seen = []
        for start in range(s.n_wgs):
            i = start
            while i >= 0 and len(seen) <= len(s.items):
                seen.append(i)
                i = s.items[i][4]
        assert sorted(seen) == list(range(len(s.items)))
    assert longest == room                  # (FULL_CHUNK: the test has seen the kernel's room used to the last word)


def _loads(s, cost):
    loads = []
    for i in range(s.n_wgs):
        loads.append(0)
        while i >= 0:
            loads[-1] += cost + s.items[i][3]
            i = s.items[i][4]
    return loads


@pytest.mark.parametrize("kind", ["latent", "latent_fp8"])
def test_latent_requests_that_need_no_cutting_are_dealt_whole(exe, kind):
    """At least a request per workgroup: the most that one gets is no more than with whole requests dealt longest first, where
    a request may be that long."""
    rng, batches = random.Random(4), []
    cost = DS.split(exe, [])[0][3 if kind == "latent" else 4]
    for n in (30, 100, 300, 1000):
        batches += [(kind, 64, cus, 1, 16, 1, 0, [int(n * (0.5 + i / (B - 1))) for i in range(B)])
                    for cus, B in ((32, 64), (32, 128), (32, 256), (64, 128), (64, 256), (128, 256))]
    batches += [(kind, P, cus, 1, 16, 1, 0, [rng.randint(1, rng.choice((20, 300, 5000))) for _ in range(rng.randint(2 * cus, 700))])
                for P in (32, 64) for cus in (32, 96) for _ in range(6)]
    _, answers = DS.split(exe, batches)
    whole_ones = 0
    for (_, P, cus, _, _, _, _, lens), s in zip(batches, answers):
        _check_cover(s.items, lens)
        heap = [0] * (2 * cus)
        for units in sorted((-(-n // TILE) for n in lens), reverse=True):
            heapq.heappush(heap, heapq.heappop(heap) + units + cost)
        whole_ones += len(s.items) == len(lens)
        assert max(_loads(s, cost)) <= max(heap) and s.n_wgs <= 2 * cus
        assert sum(_loads(s, cost)) == sum(cost + i[3] for i in s.items)          # every item in one chain
    assert 20 < whole_ones < len(batches)


def test_gqa_chunks_cover_the_batch(exe):
    batches = [("gqa", 16, cus, hkv, 64, 1, o, lens) for (lens, _, cus, o), hkv in zip(_random_batches(), [1, 2, 8, 64] * 40)]
    _, answers = DS.split(exe, batches)
    for (*_, lens), s in zip(batches, answers):
        _check_cover(s.items, lens)
        assert s.n_wgs == len(s.items) and all(i[4] == -1 for i in s.items)
        assert s.max_chunks == max(i[1] for i in s.items) + 1 and max(i[3] for i in s.items) <= s.chunk_units


LIMIT, WORKSPACE = 256 << 10, 32 << 20


def test_metadata_within_the_noalloc_limit_fits_a_staging_slot(exe):
    """The limit counts a block table row per request, the slot holds a record per work item."""
    batches = [("gqa", 16, 256, 8, 8, 0, 0, [16] * 16384),          # as many requests as the limit takes
               ("gqa", 16, 256, 8, 8, 0, 0, [9 * 16] * 5461),
               ("gqa", 16, 256, 1, 1, 0, 0, [16 * 60000]),
               ("gqa", 1024, 32, 64, 64, 0, 0, [1024 * 31] + [1] * 1900),
               ("gqa", 1024, 256, 1, 1, 0, 8, [1024 * 3800])]       # as many items as it takes, with the chunk length overridden
    batches += [("gqa", P, cus, hkv, 64, 0, o, lens) for (lens, P, cus, o), hkv in zip(_random_batches(), [1, 2, 8, 64] * 40)]
    for kind in ("noalloc", "noalloc_fp8"):
        batches += [(kind, P, cus, 1, 16, 0, o, lens) for lens, P, cus, o in _random_batches()]
        batches += [(kind, 32, 64, 1, 16, 0, 0, [32] * 16384), (kind, 64, 256, 1, 16, 1, 0, [100] * 5000)]
    (_, _, slot, *_), answers = DS.split(exe, batches)
    within = [s for s in answers if s.metadata <= LIMIT]
    assert len(within) > 200 and all(s.metadata <= LIMIT for s in answers[:5])
    assert all(s.record_bytes + 4 * 256 <= slot for s in within)    # with the largest frequency table
    assert answers[0].record_bytes > 1 << 20


# Latent batches that fit the fixed workspace with chunks of one length (of 62 pages at most), but do not as they are dealt to
# the workgroups, which cuts requests at the workgroups' borders: requests, context, page tokens, decode CUs, query heads
TIGHT = [(2187, 286, 64, 96, 7), (1179, 364, 128, 32, 14), (2598, 1339, 96, 96, 10)]
TIGHT_FP8 = [(1688, 1449, 128, 192, 11), (3608, 190, 96, 64, 8), (805, 2348, 64, 256, 14)]


@pytest.mark.parametrize("fp8,tight", [("", TIGHT), ("_fp8", TIGHT_FP8)])
def test_latent_chunks_are_lengthened_until_the_noalloc_limits_hold(exe, fp8, tight):
    _, even = DS.split(exe, [("latent" + fp8, P, cus, 1, H, 0, 0, [n] * B) for B, n, P, cus, H in tight])
    _, fit = DS.split(exe, [("noalloc" + fp8, P, cus, 1, H, 0, 0, [n] * B) for B, n, P, cus, H in tight])
    for (B, n, *_), e, f in zip(tight, even, fit):
        assert e.partials > WORKSPACE
        assert f.partials <= WORKSPACE and f.metadata <= LIMIT
        _check_cover(f.items, [n] * B)
    # a batch within the limits is split as spd_decode_step splits it
    same = [(64, 16, 1, 16, 1, 0, [1500, 65, 640, 2047])]
    assert DS.split(exe, [("noalloc" + fp8, *s) for s in same])[1][0].items == DS.split(exe, [("latent" + fp8, *s) for s in same])[1][0].items
