"""How attention launches are cut into chunks on the device (csrc/pq_decode_cut.hpp), run for the 64 lanes of a wavefront on the
CPU with the plan the host makes (csrc/pq_plan.hpp): every page of every sequence is in exactly one chunk, every chunk has one
place of the grid, its partials have rows of their own in the workspace, and each launch gets the cut it should."""
import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ON_HOST, GENERAL, GRID, FITTED = -1, 0, 1, 2
FAN = 32


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = tmp_path_factory.mktemp("cuthost") / "libcut_host.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2502_00527_amd", "csrc"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host", "cut_host.cpp"), "-o", str(out)], check=True)
    lib = ctypes.CDLL(str(out))
    lib.cut_host.restype = ctypes.c_int
    lib.cut_host.argtypes = [ctypes.c_int] * 5 + [ctypes.c_void_p, ctypes.c_int, ctypes.c_float, ctypes.c_void_p, ctypes.c_void_p]
    return lib


class Cut:
    """The cut of a launch; `chunks`: per sequence, (first page, pages) of each."""

    def __init__(self, lib, lens, kv_heads, bound=None, group=4, v_bits=16, grouped=False, error=0.0):
        bound = bound or max(lens)
        lens32 = np.asarray(lens, np.int32)
        plan = np.zeros(8, np.int64)
        slots = np.zeros((1 << 17, 6), np.int32)
        n = lib.cut_host(len(lens), kv_heads, kv_heads * group, int(grouped), v_bits, lens32.ctypes.data, bound, error, plan.ctypes.data, slots.ctypes.data)
        self.places, self.resident, self.merges, self.host_pages, self.host_chunks, self.rows, self.kind, self.used = (int(x) for x in plan)
        self.kv_heads, self.slots = kv_heads, slots[:n]
        self.pages = [(min(x, bound) + 127) // 128 if x > 0 else 0 for x in lens]
        self.chunks = [{} for _ in lens]
        self.before = {}
        for place, (seq, chunk, first, pages, n_chunks, before) in enumerate(self.slots.tolist()):
            if seq < 0:
                continue
            assert chunk not in self.chunks[seq], f"chunk {chunk} of sequence {seq} is taken twice"
            self.chunks[seq][chunk] = (first, pages, place)
            assert self.before.setdefault(seq, (n_chunks, before)) == (n_chunks, before)

    def check(self):
        assert self.used <= self.places
        assert self.merges
        at = 0
        for seq, (pages, chunks) in enumerate(zip(self.pages, self.chunks)):
            n_chunks, before = self.before[seq]
            assert sorted(chunks) == list(range(n_chunks)) and 1 <= n_chunks <= FAN, (seq, chunks)
            assert before == at, "rows of the sequences' partials, one behind the other"
            at += n_chunks
            first = 0
            for c in range(n_chunks):
                assert chunks[c][0] == first and (chunks[c][1] > 0 or pages == 0), (seq, pages, chunks)
                first += chunks[c][1]
            assert first == pages
        assert at * self.kv_heads <= self.rows, "more partials than the workspace has room for"
        return self

    def sizes(self):
        return sorted(pages for chunks in self.chunks for _, pages, _ in chunks.values())

    def rounds(self):
        """Rounds of four pages: of the fullest compute unit, if place u is on unit u % units of its KV head, and of all units in the mean."""
        units = 256 // self.kv_heads
        load = [0] * units
        for chunks in self.chunks:
            for _, pages, place in chunks.values():
                load[place % units] += (pages + 3) // 4
        return max(load), sum(load) / units


def spread(n, low, high):
    rng = random.Random(7919 * n + low + high)
    return [rng.randint(low, high) for _ in range(n)]


def draw(rng):
    kv_heads = rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 8, 8, 12, 16, 24, 32, 40, 64, 128])
    n = rng.choice([rng.randint(1, 70), rng.randint(max(1, 16 // kv_heads), 40)])
    longest = round(128 * 2 ** rng.uniform(0, 10))
    kind = rng.random()
    if kind < 0.2:
        lens = [longest] * n
    elif kind < 0.4:
        lens = [rng.randint(max(1, longest - 600), longest) for _ in range(n)]
    elif kind < 0.5:
        lens = [longest] + [rng.randint(0, 300) for _ in range(n - 1)]
    else:
        lens = [rng.randint(0, longest) for _ in range(n)]
    rng.shuffle(lens)
    bound = max(1, max(lens)) if rng.random() < 0.5 else round(max(1, max(lens)) * 2 ** rng.uniform(0, 6))
    return dict(lens=lens, kv_heads=kv_heads, bound=min(bound, 1 << 20), group=rng.choice([1, 3, 4, 8, 16]), v_bits=rng.choice([16, 4, 2]),
                grouped=rng.random() < 0.25, error=rng.choice([0.0, 2.0 ** -23, -(2.0 ** -23)]))


@pytest.mark.parametrize("seed", range(8))
def test_every_chunk_has_one_place(lib, seed):
    rng = random.Random(seed)
    seen = set()
    for _ in range(40):
        case = draw(rng)
        if case["grouped"] and case["group"] < 3:
            continue                                                   # the vector unit's kernel is cut on the host
        cut = Cut(lib, **case)
        seen.add(cut.kind)
        if cut.kind != ON_HOST:
            try:
                cut.check()
            except AssertionError:
                print(case)
                raise
    assert {GENERAL, GRID, FITTED} <= seen or len(seen) >= 3, seen


LAUNCHES = [
    # lengths, KV heads, bound, the cut on the uniform grid and with the grouped quantizer
    ([16 * 128] * 17, 8, None, GRID, GRID),
    ([700] * 20, 4, 6000, GRID, GRID),
    (spread(20, 1, 3400), 4, 3400, FITTED, FITTED),
    (spread(40, 1, 1300), 8, 1500, FITTED, FITTED),                      # more sequences than units
    ([6000] + [1 + i for i in range(40)], 2, None, FITTED, FITTED),      # units with nothing but a one-page first chunk
    (spread(23, 1, 4000), 3, 5000, FITTED, FITTED),                      # KV heads that do not divide 256
    ([0, 2900, 5, 0, 128, 129, 1000, 2432, 2433], 7, 4500, FITTED, FITTED),
    ([2300, 400], 16, 9000, FITTED, ON_HOST),                            # units without a first chunk
    (spread(63, 0, 800) + [2100], 2, 2500, FITTED, FITTED),
    (spread(48, 1000, 16000), 8, None, GENERAL, GRID),                   # chunks of 64 pages are too many to be resident together
    (spread(31, 200, 3000), 8, None, FITTED, FITTED),
    (spread(64, 1024, 16384), 8, None, GENERAL, ON_HOST),                # no places are left
    ([260] * 16, 4, 400 * 1024, GENERAL, ON_HOST),                       # the bound would have more chunks than are combined
    ([130] * 20, 2, None, ON_HOST, ON_HOST),
]


@pytest.mark.parametrize("v_bits,group,grouped", [(16, 4, False), (4, 1, False), (2, 16, False), (16, 3, True), (4, 8, True)])
@pytest.mark.parametrize("lens,kv_heads,bound,uniform,of_grouped", LAUNCHES)
def test_each_launch_gets_its_cut(lib, lens, kv_heads, bound, uniform, of_grouped, v_bits, group, grouped):
    cut = Cut(lib, lens, kv_heads, bound, group, v_bits, grouped)
    assert cut.kind == (of_grouped if grouped else uniform)
    if cut.kind != ON_HOST:
        cut.check()


@pytest.mark.parametrize("lens,v_bits", [(spread(8, 1000, 8000), 16), (spread(8, 1000, 8000), 4), (spread(16, 300, 4000), 16), (spread(16, 300, 4000), 2),
                                         (spread(32, 512, 8000), 16), (spread(32, 512, 8000), 4), (spread(4, 2000, 16000), 16)])
def test_a_loose_bound_changes_nothing(lib, lens, v_bits):
    """A serving program passes the model's context, or what a graph was captured with, for max_seq_len."""
    tight = Cut(lib, lens, 8, max(lens), v_bits=v_bits).check()
    for bound in (16384, 32768, 65536, 131072):
        cut = Cut(lib, lens, 8, bound, v_bits=v_bits).check()
        assert cut.kind == FITTED and cut.sizes() == tight.sizes() and cut.rounds() == tight.rounds(), (bound, cut.sizes(), tight.sizes())


@pytest.mark.parametrize("lens,kv_heads", [(spread(31, 750, 1500), 8), (spread(28, 96, 1530), 8), (spread(25, 1125, 1500), 8), (spread(7, 577, 1200), 32)])
def test_no_round_is_lost_to_even_chunks(lib, lens, kv_heads):
    """Two chunks of up to three rounds of four pages: 8 + 4 pages, three rounds, and not 6 + 6, four."""
    cut = Cut(lib, lens, kv_heads, 1536).check()
    assert cut.kind == FITTED
    for pages, chunks in zip(cut.pages, cut.chunks):
        assert sum((size + 3) // 4 for _, size, _ in chunks.values()) == (pages + 3) // 4, (pages, chunks)
    assert cut.rounds()[0] <= 3


@pytest.mark.parametrize("lens", [spread(48, 3000, 12000), spread(52, 3000, 12000), spread(45, 2000, 16000)])
def test_chunks_that_start_together_are_64_pages_at_most(lib, lens):
    cut = Cut(lib, lens, 8).check()
    assert max(cut.sizes()) <= 64, (cut.kind, cut.sizes())


@pytest.mark.parametrize("lens,kv_heads,bound", [([8000] * 33, 8, 8200), ([3000] * 36, 8, 3200), ([12000] * 40, 8, 12200), ([8000] * 9, 32, 8200), ([12000] * 44, 8, 12200),
                                                 ([1500] * 33, 8, 1700), ([8000] * 48, 8, 8200), ([30000] * 24, 8, 30200)])
@pytest.mark.parametrize("grouped", [False, True])
def test_places_are_not_left_empty_by_equal_sequences(lib, lens, kv_heads, bound, grouped):
    """Sequences a little shorter than the bound, a few more than compute units: not one chunk each, two of them on some units."""
    cut = Cut(lib, lens, kv_heads, bound, grouped=grouped).check()
    fullest, mean = cut.rounds()
    assert cut.kind != FITTED and max(cut.sizes()) <= 64
    assert len(cut.sizes()) > 2 * (256 // kv_heads) * 2 // 3 or max(cut.sizes()) <= 12, (cut.kind, cut.sizes())


# sequences of about the same length, a few more than compute units, or chunks of 64-page sequences that are
PAIRED = [(spread(33, 7700, 8192), 8), (spread(36, 7700, 8192), 8), (spread(40, 5800, 6100), 8), (spread(17, 7700, 8192), 16), (spread(9, 7700, 8192), 32), ([8192] * 35 + [100], 8),
          ([8192] * 20 + [600] * 13, 8), (spread(20, 7700, 8192) + spread(16, 300, 900), 8)]


@pytest.mark.parametrize("lens,kv_heads", PAIRED)
@pytest.mark.parametrize("v_bits,grouped", [(16, False), (4, False), (2, True)])
def test_no_few_units_have_two_long_chunks(lib, lens, kv_heads, v_bits, grouped):
    """More long chunks than compute units, but by less than a third: the few units with two of them would be waited for."""
    cut = Cut(lib, lens, kv_heads, v_bits=v_bits, grouped=grouped).check()
    long = sum(2 * size > max(cut.sizes()) for size in cut.sizes())
    units = 256 // kv_heads
    assert cut.kind != FITTED, (cut.sizes(), cut.rounds())
    assert len(cut.sizes()) > 2 * units * 2 // 3, (long, cut.sizes())


@pytest.mark.parametrize("lens,kv_heads,v_bits,grouped", [(spread(44, 7700, 8192), 8, 16, False), (spread(32, 512, 8192), 8, 2, False), (spread(36, 2700, 3000), 8, 4, False),
                                                          (spread(36, 1350, 1500), 8, 16, False), (spread(40, 1900, 2048), 8, 4, True), (spread(24, 7700, 8192), 8, 16, False)])
def test_all_chunks_start_at_once_where_that_is_no_slower(lib, lens, kv_heads, v_bits, grouped):
    assert Cut(lib, lens, kv_heads, v_bits=v_bits, grouped=grouped).check().kind == FITTED


@pytest.mark.parametrize("lens,v_bits", [(spread(33, 11500, 12000), 4), (spread(36, 11500, 12000), 2), (spread(33, 11500, 12000), 2), ([12000] * 34 + [12100], 4)])
def test_the_general_rule_has_the_places_it_needs(lib, lens, v_bits):
    """Quantized values, from 48 pages a resident work-group on: chunks of three quarters of a work-group's part at most."""
    cut = Cut(lib, lens, 8, v_bits=v_bits).check()
    share = (len(lens) * 8 * max(cut.pages) + 511) // 512
    assert cut.kind == GENERAL and max(cut.sizes()) <= (share * 3 // 4 + 3) // 4 * 4, (share, cut.sizes())


# Launches to which the device's first cut does not apply; tests/test_gpu_cut_fallbacks.py runs them.
# lengths, KV heads, query heads per KV head, max_seq_len, value bits, grouped quantizer, the cut
FALLBACKS = [
    (spread(33, 1690, 1790), 8, 4, 1800, 16, False, GRID),               # pairs on few units: the host's chunks
    (spread(33, 1690, 1790), 8, 1, 12100, 16, False, GENERAL),           # the same from 48 pages a resident work-group on
    (spread(17, 3700, 4090), 16, 2, 4096, 4, False, GRID),
    (spread(17, 3700, 4090), 16, 4, 12400, 2, False, GENERAL),
    (spread(9, 2200, 2430), 32, 3, 2500, 16, True, GRID),
    (spread(33, 2200, 2430), 8, 4, 12100, 4, True, GRID),                # the grouped quantizer has no general rule
    ([1700] * 33, 8, 4, 1800, 16, False, GRID),                          # equal ones below the bound
    ([1700] * 33, 8, 4, 12100, 2, False, GENERAL),
    ([1700] * 33, 8, 8, 1800, 16, True, GRID),
    ([1, 1, 1] + [1700] * 33, 8, 6, 12100, 16, False, GENERAL),
    (spread(2, 8500, 17000) + [17000], 128, 1, 17000, 4, False, GENERAL),   # chunks of 64 pages are too many
    (spread(2, 8500, 17000) + [17000], 128, 3, 17000, 2, True, GRID),
]


@pytest.mark.parametrize("lens,kv_heads,group,bound,v_bits,grouped,kind", FALLBACKS)
def test_launches_the_first_cut_does_not_apply_to(lib, lens, kv_heads, group, bound, v_bits, grouped, kind):
    cut = Cut(lib, lens, kv_heads, bound, group, v_bits, grouped).check()
    assert cut.kind == kind and cut.resident > 0, (cut.kind, cut.resident, cut.sizes())
