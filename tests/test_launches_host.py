"""Every rule by which the library chooses and sizes its launches, on the CPU: the launchers are compiled for
the host only against a HIP runtime that records launches (launches.py), and each recorded launch is checked for
what the runtime accepts, for covering its range exactly, and for keeping its partials inside the workspace."""
from __future__ import annotations

import random

import pytest

from kernel_calls import BEGIN, CALLS
from launches import FAR, FULL, MIN_WS, NEAR, NEAR16, WORK, Recorder, build, check, parse_name, shape

STEPS = ["step", "oop", "from_acc", "host_step"]
NORMS = ["norm", "staged", "acc_norm", "add_norm", "spec", "noalloc"]
ENTRIES = STEPS + ["add"] + NORMS


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    return Recorder(build(str(tmp_path_factory.mktemp("launches"))))


# HIP launches fewer than 2^32 work items at a time: with 2 elements per lane that is less than 2^33 elements,
# with 4 less than 2^34.  A 309 GB card holds the staged step's 18 bytes per element up to 1.7e10 elements.
@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("length", [(1 << 33) - 1025, (1 << 33) - 1, 1 << 33, (1 << 33) + 1, (1 << 34) - 1024, (1 << 34) - 257])
@pytest.mark.parametrize("begin", [0, 5])
def test_longest_ranges_are_launched(rec, entry, length, begin):
    for k in (1, 4, 8, 16, 32):
        for ws in (MIN_WS, FULL):
            for cus in (256, 64):
                if entry == "noalloc" and length > 1 << 33:
                    continue
                st, launches, _, wsb = rec.call(entry, k, begin, begin + length, ws, cus=cus)
                assert st == 0, (entry, k, ws, cus, [l.name for l in launches])
                check(entry, launches, begin, begin + length, wsb)


def _lengths(rng):
    for p in range(0, 33):
        yield rng.randrange(1 << p, 2 << p)
    for line in (1 << 18, 1 << 19, 960_000, 1_400_000, 3 << 19, 1 << 21, 7_000_000, 1 << 22, 1 << 23, 1 << 24, 1 << 25, 3 << 24, 1 << 26,
                 1 << 27, 1 << 28, 1 << 29):
        yield from (line - 1, line, line + 1)


@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("seed", [0, 1])
def test_launches_cover_any_range(rec, entry, seed):
    rng = random.Random(seed)
    for length in _lengths(rng):
        for k in [1, 2, 3, 4, 5, 7, 8, 9, rng.randint(10, 32)]:
            begin = rng.choice([0, 1, 2, 3, 4, 1023, 4096, rng.randrange(1 << 20), rng.randrange(1 << 33)])
            ws = rng.choice([MIN_WS, FULL, MIN_WS + 8 * rng.randrange(1 << 20)])
            st, launches, _, wsb = rec.call(entry, k, begin, begin + length, ws, accumulate=rng.randrange(2),
                                            first=rng.randrange(2), cus=rng.choice([16, 128, 256]))
            assert st == 0
            check(entry, launches, begin, begin + length, wsb)


@pytest.mark.parametrize("entry", NORMS)
@pytest.mark.parametrize("begin", [0, 5, 4096])
def test_empty_range_writes_a_zero_norm(rec, entry, begin):
    for k in (1, 5):
        st, launches, _, wsb = rec.call(entry, k, begin, begin)
        assert st == 0
        check(entry, launches, begin, begin, wsb)
        st, launches, _, _ = rec.call(entry, k, begin, begin, accumulate=1)
        assert st == 0 and not launches


# hipStreamLegacy and hipStreamPerThread are names of streams, not streams: nothing but a launch is given them
@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("stream", [0, 1, 2])
def test_cus_of_the_special_streams_are_not_asked_for(rec, entry, stream):
    for length in (1000, 3_000_000, 100_000_000):
        for k in (1, 8):
            st, launches, asked, _ = rec.call(entry, k, 0, length, cus=64, stream=stream)
            assert st == 0 and not asked
            plain = rec.call(entry, k, 0, length, cus=256)[1]
            assert [(l.name, l.grid) for l in launches] == [(l.name, l.grid) for l in plain]     # as on all CUs


def work_of(rec, *args, **kw):
    """The launch that does the work of a call (the others fold partials)."""
    return rec.call(*args, **kw)[1][0]


# streams confined to some of the CUs: the limit of the norm's long runs is one of elements per CU
@pytest.mark.parametrize("k", [1, 3, 4, 5, 7, 8, 16])
def test_norm_on_some_of_the_cus(rec, k):
    for cus in (16, 64, 128, 256):
        for per_cu in (40_000, 49_152, 98_304, 1_000_000):
            n = per_cu * cus
            l = work_of(rec, "norm", k, 3, 3 + n, cus=cus)
            long_runs = 4 <= k <= 7 and cus < 256 and per_cu >= (98_304 if k == 4 else 49_152) and n > 1 << 19
            assert (l.targs == (0, 1, 256, 0, 4) and l.extra == 8) == long_runs, (cus, per_cu, l.name)


def first_kept(l, keep_from):
    """The first element of the first workgroup that starts at keep_from or beyond."""
    block, el, _ = shape(l)
    run = block * el * l.extra
    base = l.begin // (block * el) * block * el
    return max(l.begin, base + -(-(keep_from - base) // run) * run)


def held(l, declared=0):
    """Workgroups of a launch that a CU holds by its LDS, which is handed out in 128 pieces of 1280 bytes."""
    assert l.lds + declared <= 65536
    return 128 // -(-(l.lds + declared) // 1280) if l.lds else None


# CUs of the stream: workgroups a CU holds (None: no bound).  A die's share is what its least shader engine makes of
# it; where the dies' shares differ (18, 20, 28, 60, 92 CUs) nothing is held back
@pytest.mark.parametrize("cus,want", [(8, 21), (16, 11), (18, None), (20, None), (24, 7), (28, None), (32, 5), (36, 5), (40, 5), (48, 5), (56, 5),
                                      (60, None), (64, 2), (72, 2), (88, 2), (92, None), (96, 5), (120, 5), (124, None), (128, 4), (136, 4),
                                      (160, 3), (192, 3), (224, 2), (255, None), (256, 2)])
def test_step_on_host_memory_keeps_as_many_waves_in_flight_as_the_link_needs(rec, cus, want):
    for k in (1, 4, 8, 9, 16, 32):
        for length in (1, 1000, 300_000, 12_600_000, 800_000_000):
            l = work_of(rec, "host_step", k, 3, 3 + length, cus=cus)
            assert l.targs == (64, 2, 0, 16 if k > 8 else 8, 0, 0, 1, 0) and held(l) == want, (k, length, l.name, l.lds)


# a step above 2^21 elements: (loads in flight, workgroups a CU holds)
def long_step(k, length):
    if length <= 7_000_000:
        return (8, None) if 5 <= k < 20 else (4, None)
    stream, deep = (4, 10 if k % 4 == 0 else 11), (8, 9)
    if k < 5 or k > 24:
        return stream
    if k < 8:
        return deep
    if k % 8 == 0:
        return deep if length <= 1 << 25 else stream
    if length <= 1 << 24:
        return 4, None
    return deep if k < 20 and length <= 1 << 26 else stream


def test_long_steps_hold_as_many_workgroups_as_meant(rec):
    for length in ((1 << 21) + 1, 7_000_000, 7_000_001, 1 << 24, (1 << 24) + 1, 1 << 25, (1 << 25) + 1, 1 << 26, (1 << 26) + 1, 800_000_000):
        for k in range(1, 33):
            depth, workgroups = long_step(k, length)
            for entry in ("step", "oop"):
                l = work_of(rec, entry, k, 3, 3 + length)
                assert l.targs == (128, 2, 0, depth, 0, 0, 1, 0) and held(l) == workgroups, (k, length, l.name, l.lds)
            l = work_of(rec, "step", k, 3, 3 + length, cus=64)
            assert l.targs == (64, 4, 0, 2, 0, 1, 0, 0) and l.lds == 0
        l = work_of(rec, "from_acc", 1, 3, 3 + length)
        short = length <= 7_000_000
        assert l.targs == ((128, 2, 1, 4, 0, 0, 1, 0) if short else (64, 4, 1, 4, 0, 0, 1, 0)) and held(l) == (None if short else 10)


@pytest.mark.parametrize("ws", [MIN_WS, FULL])
def test_speculative_pass_holds_as_many_workgroups_as_meant(rec, ws):
    for length in (1000, 1 << 21, (1 << 21) + 1, 7_000_000, 7_000_001, 67_000_000, 67_200_000, 134_000_000, 134_300_000, (1 << 28) - 1, 1 << 28,
                   (1 << 29) - 1, 1 << 29):
        for k in range(1, 33):
            l = work_of(rec, "spec", k, 3, 3 + length, ws)
            if length <= 7_000_000:
                want, workgroups = (256, 4, 16, 0, int(k <= 2 or (k <= 7 and length <= 1 << 21))), None
            elif ws == FULL or length <= 67_000_000:
                want, workgroups = (64, 4, 4, 0, 1), 16 if k <= 8 else 14
            elif length <= 134_000_000:
                want, workgroups = (128, 4, 4, 0, 1), 8 if k <= 4 else 7
            elif length < (1 << 28 if k <= 2 else 1 << 29):
                want, workgroups = (256, 2, 4, 0, 1), 6 if length < 1 << 28 else 5
            else:
                want, workgroups = (1024, 4, 8, 0, 1), None
            assert l.targs == want and held(l, declared=l.block // 64 * 8) == workgroups, (k, length, l.name, l.lds)


def test_nothing_else_keeps_workgroups_off_a_cu(rec):
    for entry in ("add", "norm", "noalloc", "staged", "acc_norm", "add_norm"):
        for length in (1000, 1 << 20, 12_600_000, 500_000_000):
            for k in (1, 3, 8, 16, 32):
                assert all(l.lds == 0 for l in rec.call(entry, k, 3, 3 + length)[1])


@pytest.mark.parametrize("cus", [16, 128, 256])
def test_norm_of_one_stream_takes_runs_of_eight_where_the_fold_counts(rec, cus):
    for length in (1 << 22, (1 << 23) - 1, 1 << 23, 3 << 24, (3 << 24) + 1, 1 << 26, 1 << 28, (1 << 29) - 1, 1 << 29, 1 << 30):
        l = work_of(rec, "norm", 1, 3, 3 + length, ws=FULL, cus=cus)
        long_run = length >= 1 << 23 and (length <= 3 << 24 or length >= 1 << 29 or cus < 256)
        assert l.targs[:3] == (1, 4, 256) and l.extra == (8 if long_run else 4), length


def test_step_in_full_cus_has_eight_loads_in_flight_up_to_19_streams(rec):
    for k in range(1, 33):
        for length in ((1 << 21) + 1, 4_000_000, 7_000_000):
            l = work_of(rec, "step", k, 3, 3 + length)
            assert l.targs == (128, 2, 0, 8 if 5 <= k < 20 else 4, 0, 0, 1, 0) and l.lds == 0, (k, length, l.name)


@pytest.mark.parametrize("cus", [64, 256])
def test_later_micro_batches_of_a_small_range_stay_in_the_cache(rec, cus):
    for length in (1, 13_000, 1 << 20, 1 << 21, (1 << 21) + 1, 1 << 22, (1 << 22) + 1, 100_000_000):
        l = work_of(rec, "add", 1, 5, 5 + length, cus=cus)
        waits = length > 1 << 22 and cus == 256
        assert l.targs == (0, 0, 64, 4, waits, length > 1 << 21), (length, l.name)
        assert work_of(rec, "add", 1, 5, 5 + length, first=1, cus=cus).targs[-1] == 0
        assert work_of(rec, "add_norm", 1, 5, 5 + length, cus=cus).targs[-1] == 0


def test_step_of_a_small_range_writes_through_while_its_loads_last(rec):
    for k in range(1, 33):
        upto = 0 if k == 1 or k >= 16 else 1 << 19 if k < 5 else 1 << 18 if k == 8 else (1 << 19) - 12_000 * k
        for length in (1, 100_000, 1 << 18, (1 << 18) + 1, upto, upto + 1, 1 << 19):
            if not 1 <= length <= 1 << 19:
                continue
            for cus in (16, 256):
                l = work_of(rec, "step", k, 3, 3 + length, cus=cus)
                assert l.targs == (64, 2, 0, 16 if k > 8 else 8, 0, 0, length <= upto, 0) and l.lds == 0, (k, length, l.name)


def test_step_of_one_generation_reads_its_arguments_late_while_the_memory_is_busy(rec):
    for k in range(1, 33):
        for cus in (64, 256):
            for length in ((1 << 19) + 1, 960_000, 960_001, 1_100_000, 1_100_001, 1_240_001, 1_380_000, 1_400_000, 1_400_001, 3 << 19, (3 << 19) + 1, 1 << 21):
                above = {4: 1_380_000, 5: 1_240_000, 6: 1_100_000}.get(k, 960_000)
                upto = 3 << 19 if k == 4 else 1 << 21 if k < 8 else 1_400_000
                late = k >= 4 and above < length <= upto and cus == 256
                serial = k <= 7 and length > 3 << 19
                for entry in ("step", "oop"):
                    l = work_of(rec, entry, k, 0, length, cus=cus)
                    assert l.targs == (64, 4, 0, *((1, 1, 1) if serial else (4, 0, 1)), 0, late), (k, length, cus, l.name)
                l = work_of(rec, "from_acc", 1, 0, length, cus=cus)
                assert l.targs[2] == 1 and l.targs[-1] == 0


def takes_distances(k, length, cus):
    """Whether a step in place, all of whose arrays lie near p, is given them by their distances."""
    if k > 8:
        return False
    if length <= 1 << 19:
        return length <= (430_000 if k in (1, 8) else 330_000 - 9_000 * k)
    if length <= 1_200_000:
        return cus < 256 or length <= {6: 1_100_000, 7: 960_000, 8: 960_000}.get(k, 1_200_000)
    return 1 << 21 < length <= 5_000_000 and cus == 256


NEAR_LINES = [1, 1001, 1 << 18, *(330_000 - 9_000 * k for k in range(2, 8)), 430_000, 1 << 19, 960_000, 1_100_000, 1_200_000, 3 << 19, 1 << 21,
              5_000_000, 7_000_000, 12_600_000]


@pytest.mark.parametrize("k", range(1, 10))
@pytest.mark.parametrize("cus", [64, 256])
def test_step_in_place_is_given_distances(rec, k, cus):
    for length in sorted({n + d for n in NEAR_LINES for d in (0, 1)}):
        for begin in (0, 3):
            for at, near in ((NEAR, True), (NEAR16, True), (FAR, False)):
                for more in ({}, {"sqnorm": False}, {"max_norm": 0.0}):
                    consts = work_of(rec, "oop", k, begin, begin + length, **more).consts
                    st, launches, _, wsb = rec.call("step", k, begin, begin + length, cus=cus, at=at, **more)
                    assert st == 0
                    check("step", launches, begin, begin + length, wsb, at)
                    assert launches[0].consts == consts and len(set(consts)) > 7
                    assert launches[0].near == (near and takes_distances(k, length, cus)), (k, length, cus, launches[0].name)
            for entry in ("oop", "from_acc"):
                assert not work_of(rec, entry, k, begin, begin + length, cus=cus, at=NEAR).near


@pytest.mark.parametrize("name", ["p", "m", "v", "w", "g0", "g3", "g4", "g7"])
def test_step_with_an_array_too_far_away_is_given_addresses(rec, name):
    """A distance is 32 bits of 256 bytes if all of them are multiples of that, else of 16."""
    for at, unit in ((NEAR, 256), (NEAR16, 16)):
        for length in (1, 1001, 200_000, 600_001, (1 << 21) + 1):
            for distance in (-(1 << 31) - 1, -(1 << 31), (1 << 31) - 1, 1 << 31):
                other = at.m if name == "p" else getattr(at, name) if name[0] != "g" else at.g[int(name[1:])]
                by = distance * unit + (other - at.p if name == "p" else at.p - other)
                moved = at.moved(name, by)
                l = work_of(rec, "step", 8, 3, 3 + length, at=moved)
                fits = all(-(1 << 31) <= (x - moved.p) // unit < 1 << 31 for x in (moved.m, moved.v, moved.w, *moved.g[:8]))
                assert l.near == fits, (length, unit, distance)
                assert fits or name == "p" or distance not in (-(1 << 31), (1 << 31) - 1)
    # one array off the multiples of 256: the unit is 16 for all of them
    assert not work_of(rec, "step", 8, 0, 1001, at=NEAR.moved(name, 16).moved("v" if name != "v" else "m", 1 << 36)).near


@pytest.mark.parametrize("k", range(1, 33))
def test_norm_leaves_its_last_lines_in_the_cache(rec, k):
    line = 1 << 21 if k == 1 else 1_300_000 if k < 4 else 3 << 18
    for length in (1, 20_000, 1 << 19, line, line + 1, (1 << 21) + 1, 5_500_001, 12_600_000, 300_000_000):
        for cus, accumulate in ((256, 0), (256, 1), (64, 0)):
            for ws in (MIN_WS, FULL):
                l = work_of(rec, "norm", k, 5, 5 + length, ws=ws, cus=cus, accumulate=accumulate)
                keeps = length > line and cus == 256 and not accumulate
                assert l.keep_from == (first_kept(l, 5 + length - (1 << 28) // (2 * k)) if keeps else 5 + length), (length, cus, accumulate)


# on a stream confined to some of the CUs the bytes that each of them has in flight are what counts
@pytest.mark.parametrize("cus", [16, 64, 128, 192])
def test_speculative_pass_on_some_of_the_cus_fills_them(rec, cus):
    for k in (1, 2, 7, 8, 11, 16, 32):
        for length in ((1 << 21) + 1, 12_600_000, 67_000_000, 67_200_000, 134_000_000, 134_300_000, (1 << 28) - 1, 1 << 28, 1 << 29, 1 << 32):
            for ws in (MIN_WS, FULL):
                l = work_of(rec, "spec", k, 3, 3 + length, ws, cus=cus)
                assert l.lds == 0, (k, length, l.name)
                # a partial per 256 elements; per 512, and up to 2^28 elements with few streams in runs; runs of as many
                want = (64, 4, 2, 1, 0) if ws == FULL or length <= 67_000_000 else \
                    (128, 4, 4, 1, 0) if length <= 134_000_000 or (k <= 7 and length < 1 << 28) else (256, 2, 4, 0, 1)
                assert l.targs == want, (k, length, l.name)


def test_staged_norm_of_long_ranges_pairs_elements_for_whole_batches_only(rec):
    for length in ((1 << 25) - 1, 1 << 25, 200_000_000):
        for k in range(1, 33):
            for cus in (64, 256):
                l = work_of(rec, "staged", k, 0, length, ws=FULL, cus=cus)
                pairs = length >= 1 << 25 and k >= 8 and k % 4 == 0 and cus == 256
                assert l.targs[:3] == ((256, 2, 4) if pairs else (64, 4, 2) if k <= 8 else (128, 4, 2)), (length, k, cus)


def test_staged_norm_keeps_its_sum_cached_for_few_streams_only(rec):
    for length in (1 << 21, (1 << 21) + 1, 12_600_000, 200_000_000):
        for k in range(1, 33):
            for cus, accumulate in ((256, 0), (256, 1), (64, 0)):
                l = work_of(rec, "staged", k, 5, 5 + length, ws=FULL, cus=cus, accumulate=accumulate)
                keeps = k <= 16 and length > 1 << 21 and cus == 256 and not accumulate
                assert l.keep_from == (first_kept(l, 5 + length - (64 << 20)) if keeps else 5 + length)
                assert l.targs[3] == keeps


def test_staged_norm_takes_wide_workgroups_in_the_middle(rec):
    for k in range(1, 33):
        for cus in (16, 64, 256):
            for length in ((1 << 19) + 1, 40_000 * cus, 49_152 * cus, 1 << 20, (1 << 20) + 1, 3_300_000, 1 << 22, (1 << 22) + 1):
                if length <= 1 << 19:
                    continue
                l = work_of(rec, "staged", k, 0, length, ws=FULL, cus=cus)
                wide = length <= (1 << 22 if k <= 16 else 1 << 20) and not (cus < 256 and k < 8 and length >= 49_152 * cus)
                assert l.targs[:3] == ((1024, 4, 4) if wide else (64, 4, 2) if k <= 8 else (128, 4, 2)), (k, cus, length)


def test_staged_norm_with_a_small_workspace(rec):
    for length in (1 << 27, (1 << 27) + 1, 500_000_000, 1 << 32):
        for k in range(1, 33):
            l = work_of(rec, "staged", k, 0, length, ws=MIN_WS)
            if length > 1 << 27:                   # no room for a partial per 512 elements
                assert l.targs[:3] == ((128, 4, 2) if k <= 3 else (1024, 4, 2))


def test_the_gpu_tests_calls_reach_every_kernel(rec):
    """test_gpu_kernels.py runs every kernel of the library, and the library holds none that no call reaches."""
    names = {parse_name(n) for n in rec.kernels()}
    reached = set()
    for entry, k, length, ws, cus, first, accumulate in CALLS:
        st, launches, _, _ = rec.call(entry, k, BEGIN, BEGIN + length, FULL if ws == "full" else MIN_WS, accumulate=accumulate, first=first, cus=cus, at=NEAR)
        assert st == 0
        reached |= {(l.kernel, l.targs, l.params) for l in launches}
    assert names - reached == set()                # the two folds too
    assert reached - names == set()
