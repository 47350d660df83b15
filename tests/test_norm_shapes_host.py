"""The norm's shapes from five streams on, by length, on the CPU: the launchers against a HIP runtime that records launches."""
from __future__ import annotations

import pytest

from launches import FULL, MIN_WS, Recorder, build, check


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    return Recorder(build(str(tmp_path_factory.mktemp("launches"))))


@pytest.mark.parametrize("k", range(5, 33))
def test_norm_has_a_kernel_for_each_number_of_streams(rec, k):
    for length, lanes, tiles in ((1, 1024, 1), (4096, 1024, 1), (4097, 256, 1), (3 << 18, 256, 1), ((3 << 18) + 1, 512, 1), (5_500_000, 512, 1),
                                 (5_500_001, 1024 if k < 8 else 512, 2), (1 << 25, 1024 if k < 8 else 512, 2), ((1 << 25) + 1, 512, 2),
                                 ((1 << 29) - 1, 512, 2), (1 << 29, 512, 4)):
        for ws in (MIN_WS, FULL):
            for begin in (0, 5):
                one = length + begin % 4096 <= 4096
                st, launches, _, wsb = rec.call("norm", k, begin, begin + length, ws)
                assert st == 0
                check("norm", launches, begin, begin + length, wsb)
                l = launches[0]
                if one:
                    lanes_, tiles_ = 1024, 1
                else:
                    lanes_, tiles_ = (256, 1) if length <= 4097 else (lanes, tiles)
                assert l.targs == (k, 1, lanes_, one, 16), (length, l.name)
                assert l.extra == tiles_ or ws == MIN_WS, (length, l.extra)


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
