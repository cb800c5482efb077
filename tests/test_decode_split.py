"""Host logic, no GPU: every tile of a decode batch belongs to one chunk, chains of chunks are walks through all of them, and
no chunk of the latent decode touches more pages than its kernel has room for."""
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


def test_latent_chunks_fit_the_kernel(exe):
    batches = [("latent", P, cus, 1, 0, [n] * B) for B, n, P, cus in LONG]
    batches += [("latent", P, cus, 1, o, lens) for lens, P, cus, o in _random_batches()]
    room, words, answers = DS.split(exe, batches)
    assert room + words <= KERNEL_THREADS
    longest = 0
    for (_, P, cus, _, override, lens), (n_wgs, max_chunks, chunk_units, items) in zip(batches, answers):
        per_page = P // TILE
        most = max(_pages(u0, n, per_page) for _, _, u0, n, _ in items)
        longest = max(longest, most)
        assert most <= room, (P, cus, len(lens), most)
        # the record as the host lays it out
        assert min(-(-max(lens) // P), (chunk_units + per_page - 2) // per_page + 1) <= room
        _check_cover(items, lens)
        assert max_chunks == max(c for _, c, _, _, _ in items) + 1 and chunk_units == max(n for _, _, _, n, _ in items)
        assert override or n_wgs <= 2 * cus
        # the chains that workgroups 0 .. n_wgs - 1 walk pass through every item once
        seen = []
        for start in range(n_wgs):
            i = start
            while i >= 0 and len(seen) <= len(items):
                seen.append(i)
                i = items[i][4]
        assert sorted(seen) == list(range(len(items)))
    assert longest == room                  # (FULL_CHUNK: the test has seen the kernel's room used to the last word)


def test_gqa_chunks_cover_the_batch(exe):
    batches = [("gqa", 16, cus, hkv, o, lens) for (lens, _, cus, o), hkv in zip(_random_batches(), [1, 2, 8, 64] * 40)]
    _, _, answers = DS.split(exe, batches)
    for (_, _, cus, hkv, override, lens), (n_wgs, max_chunks, chunk_units, items) in zip(batches, answers):
        _check_cover(items, lens)
        assert n_wgs == len(items) and all(i[4] == -1 for i in items)
        assert max_chunks == max(c for _, c, _, _, _ in items) + 1 and max(n for _, _, _, n, _ in items) <= chunk_units
