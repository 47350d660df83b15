"""Calls that between them reach every kernel of the library and both sides of the lines that the launchers draw
for long ranges.  test_launches_host.py checks on the CPU that they do; test_gpu_kernels.py runs them.

(entry point as in launches.py, streams, length of the range, "min" or "full" workspace, CUs of the stream (256: an
ordinary one), first micro-batch, accumulate onto an earlier norm)"""
L19, L20, L21, L22, L23, L25, L27, L28 = (1 << p for p in (19, 20, 21, 22, 23, 25, 27, 28))


def _c(entry, k, length, ws="min", cus=256, first=0, accumulate=0):
    return entry, k, length, ws, cus, first, accumulate


CALLS = [
    # the step with its arrays by distances, a kernel for each number of streams: arrays of one training program lie near enough
    *[_c("step", k, n) for k in range(1, 9) for n in (1001, 600_001, L21 + 1)], _c("step", 8, 300_001),
    # the step given addresses, in place and out of place, and the staged step, by length and on some of the CUs
    *[_c("oop", k, n) for k, n in ((1, 1), (2, 1), (5, 3), (6, 500_000), (1, L19 + 1), (7, L21 + 1), (2, L21 + 1))],
    *[_c("step", k, n) for k, n in ((1, 1), (2, 1), (5, 3), (9, 1), (17, 1001), (6, 500_000), (12, 500_000), (1, L19 + 1), (3, 1_600_000), (7, L21 + 1), (13, 7_000_001),
                                    (6, L27 + 1), (10, L27 + 1))],
    *[_c("step", k, L21 + 1, cus=64) for k in (1, 5)],
    *[_c("step", k, n) for k, n in ((4, 1_380_001), (6, 1_100_001), (9, 1_400_000), (9, 1_400_001), (7, 1_600_000))],
    *[_c("from_acc", 1, n) for n in (1, L19 + 1, 1_600_000, L21 + 1, 7_000_001, L27 + 1)],
    _c("from_acc", 1, L21 + 1, cus=64),
    # the speculative pass: by length, workspace and streams left over after batches of four; a long range and the lines
    # with a small workspace, at a partial per 256 or 512 elements and at 2^28 elements; on some of the CUs
    *[_c("spec", k, n) for k, n in ((1, 1), (5, 1001), (16, 7_000_000), (1, L19 + 1), (2, 7_000_001))],
    *[_c("spec", k, 7_000_001, "full") for k in (3, 4, 5, 6, 12, 13, 14, 15)],
    *[_c("spec", k, n, "full") for k in (3, 8) for n in (79_999_999, 80_000_000)],
    *[_c("spec", k, n) for k in (2, 3, 9) for n in (66_000_000, 67_200_000, L27 - 20_000, L27 + 1)],
    *[_c("spec", k, n) for k in (2, 7, 8, 11) for n in (L28 - 1, L28)],
    _c("spec", 1, L21 + 1, cus=64),
    *[_c("spec", k, n, cus=64) for k, n in ((6, 67_200_000), (7, 134_300_000), (9, 134_300_000))],
    # the norm: one workgroup, then by length for each number of streams with a kernel of its own; from
    # five on in 256 and 512 lanes, up to seven in 1024; long runs on some of the CUs
    *[_c("norm", k, n) for k in (1, 2, 3, 4) for n in (1, 16_000, 20_000, L22, L22 + 1)],
    *[_c("norm", k, n) for k in (5, 8, 23) for n in (1, 5000, L20, L20 + 1, L21, L21 + 1, L23, L23 + 1)],
    *[_c("norm", k, n) for k in range(5, 33) for n in (1, 5000, 20_000, L20)], *[_c("norm", k, 6_000_000) for k in (5, 6, 7)],
    *[_c("norm", k, 1_000_000, cus=16) for k in (5, 7)], _c("norm", 4, 6_400_000, cus=64),
    _c("norm", 8, 12_600_000, accumulate=1),
    # the norm of an fp32 sum
    *[_c("acc_norm", 1, n) for n in (1, 20_000, L22 + 1, L27 - 1, L27 + 1)],
    # the staged norm: by length, streams, workspace and CUs; with and without the sum's end left in the cache
    *[_c("staged", k, n) for k, n in ((1, 1), (8, 1), (3, L19 + 1), (17, L20), (17, L20 + 1), (7, L21 + 1), (1, L22 + 1), (9, L22 + 1), (20, L22 + 1))],
    *[_c("staged", k, n) for k, n in ((9, 1001), (9, 5_000_001), (12, L25))], _c("staged", 9, L27 + 1, accumulate=1),
    _c("staged", 2, L22 + 1, accumulate=1), _c("staged", 9, L22 + 1, accumulate=1), _c("staged", 2, 1_000_000, cus=16),
    *[_c("staged", k, n) for k in (8, 9) for n in (L25 - 1, L25)],
    _c("staged", 8, L25, accumulate=1), _c("staged", 20, L25),
    *[_c("staged", k, n) for k in (1, 3, 4, 5, 9) for n in (L27 - 20_000, L27 + 1)],
    _c("staged", 4, L27 + 1, accumulate=1), _c("staged", 2, L27 + 1, accumulate=1),
    # adding a micro-batch, without and with the norm
    *[_c("add", 1, n, first=f) for f in (0, 1) for n in (1, L22, L22 + 1)],
    _c("add", 1, L21 + 1), _c("add", 1, L22 + 1, cus=64), *[_c("add", 1, n, first=1) for n in (900_000, 900_001, L21, L21 + 1, L25, L25 + 1)],
    *[_c("add_norm", 1, n, first=f, accumulate=a) for n in (L21, L21 + 1, L22, L22 + 1) for f in (0, 1) for a in (0, 1)],
    *[_c("add_norm", 1, n, first=f) for f in (0, 1) for n in (1, L19, L19 + 1, L23, L23 + 1)],
    *[_c("add_norm", 1, n) for n in (67_200_000, L28 + 1)],
]
BEGIN = 5          # of every range: ragged at both ends
