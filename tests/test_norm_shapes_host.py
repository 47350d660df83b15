"""The norm's shapes from five streams on, by length, on the CPU: the launchers against a HIP runtime that records launches."""
from __future__ import annotations

import pytest

from launches import FULL, MIN_WS, Recorder, build, check


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    return Recorder(build(str(tmp_path_factory.mktemp("launches"))))


@pytest.mark.parametrize("k", range(5, 33))
def test_norm_has_a_kernel_for_each_number_of_streams(rec, k):
    for length, lanes, tiles in ((1, 1024, 1), (4096, 1024, 1), (4097, 256, 1), (65536 // k, 256, 1), (65536 // k + 1, 256, 1), (3 << 18, 256, 1), ((3 << 18) + 1, 512, 1), (5_500_000, 512, 1),
                                 (5_500_001, 1024 if k < 8 else 512, 2), (1 << 25, 1024 if k < 8 else 512, 2), ((1 << 25) + 1, 512, 2),
                                 ((1 << 29) - 1, 512, 2), (1 << 29, 512, 4)):
        for ws in (MIN_WS, FULL):
            for begin in (0, 5):
                spanned = (begin + length - 1) // 4096 + 1
                one = spanned == 1 or length * k <= 65536
                st, launches, _, wsb = rec.call("norm", k, begin, begin + length, ws)
                assert st == 0
                check("norm", launches, begin, begin + length, wsb)
                l = launches[0]
                if one:
                    lanes_, tiles_ = 1024, spanned
                else:
                    lanes_, tiles_ = (256, 1) if length <= 65536 else (lanes, tiles)
                assert l.targs == (k, 1, lanes_, one, 16), (length, l.name)
                assert l.extra == tiles_ or ws == MIN_WS, (length, l.extra)


@pytest.mark.parametrize("entry", ["norm", "noalloc"])
@pytest.mark.parametrize("k", range(5, 33))
def test_captured_norm_is_left_to_one_workgroup_where_its_gpu_time_is_less(rec, entry, k):
    for begin in (0, 4, 5, 13, 1021, 4093):
        for length in (1, 4096 - begin % 4096, 4097, 40960 // k, 40960 // k + 1, 65536 // k, 65536 // k + 1, 8192, 8200 - begin, 100_000):
            end, tiles = begin + length, (begin + length - 1) // 4096 - begin // 4096 + 1
            in_one_wave = begin % 4 and end % 4 and begin % 4096 // 256 == end % 4096 // 256
            for capturing in (False, True):
                st, launches, _, wsb = rec.call(entry, k, begin, end, capturing=capturing)
                assert st == 0
                check(entry, launches, begin, end, wsb)
                if capturing:
                    one = length * k <= 40960 and tiles == -(-length // 4096) and not in_one_wave
                else:
                    one = length * k <= 65536
                assert launches[0].targs[3] == (one or tiles == 1), (begin, length, capturing)
            # the null stream is not captured and not asked about
            assert rec.call(entry, k, begin, end, capturing=True, stream=0)[1][0].targs[3] == (length * k <= 65536 or tiles == 1)


@pytest.mark.parametrize("k", [1, 8, 16, 17, 32])
def test_staged_norm_takes_wide_workgroups_again(rec, k):
    for length in ((1 << 22) + 1, 4_499_999, 4_500_000, 10_000_000, 10_000_001, 12_600_000):
        for cus in (64, 256):
            for ws in (MIN_WS, FULL):
                st, launches, _, wsb = rec.call("staged", k, 5, 5 + length, ws, cus=cus)
                assert st == 0
                check("staged", launches, 5, 5 + length, wsb)
                wide = k <= 16 and 4_500_000 <= length <= 10_000_000 and cus == 256
                assert launches[0].targs[:3] == ((1024, 4, 4) if wide else (64, 4, 2) if k <= 8 else (128, 4, 2)), (length, cus)


@pytest.mark.parametrize("cus", [64, 256])
def test_adding_kernel_by_length(rec, cus):
    all_cus = cus == 256
    for length in (1, 900_000, 900_001, 1 << 21, (1 << 21) + 1, 1 << 22, (1 << 22) + 1, 1 << 23, (1 << 23) + 1, 60_000_000):
        l = rec.call("add", 1, 5, 5 + length, first=1, cus=cus)[1][0]
        lanes = 256 if length <= 900_000 or not all_cus else 512 if length <= 1 << 21 else 128 if length <= 1 << 25 else 64
        assert l.targs == (1, 0, lanes, 4, 0, 0), (length, l.name)
        for first in (0, 1):
            for accumulate in (0, 1):
                st, launches, _, wsb = rec.call("add_norm", 1, 5, 5 + length, first=first, accumulate=accumulate, cus=cus)
                assert st == 0
                check("add_norm", launches, 5, 5 + length, wsb)
                l = launches[0]
                keeps = length > (1 << 23 if first else 1 << 22) and all_cus and not accumulate
                assert (l.keep_from < l.end) == keeps, (length, first, accumulate)
                lanes = 256 if length <= 1 << 19 else 64 if keeps or length > 1 << 23 else 1024
                assert l.targs == (first, 1, lanes, 4, 0, 0), (length, first, accumulate, l.name)
