"""The kernel that a call is planned on, for the calls of the GPU tests: those that mean to test one of the kernels reach it.
No GPU is used."""
import pytest

import paper_2503_01873_amd as P
from gpu_harness import plan_of, row_blocks_of

MSD = (P.MIXED, P.S16, P.DIRECT)


@pytest.mark.parametrize("B,Hq,Hkv,Nq,row0,N,d,causal,variants,kernel,split", [
    # test_few_rows
    (2, 2, 2, 1, 0, 1, 128, True, MSD, "rows", False),
    (2, 14, 2, 1, 62, 63, 64, True, MSD, "rows", False),
    (2, 16, 2, 2, 62, 64, 128, True, MSD, "rows", False),
    (2, 14, 2, 3, 62, 65, 64, True, MSD, "rows", False),
    (2, 6, 2, 15, 600, 1025, 64, True, MSD, "rows", False),
    (2, 4, 2, 16, 624, 640, 128, True, MSD, "rows", False),
    (2, 4, 2, 17, 0, 513, 64, True, MSD, "rows", False),
    (2, 2, 2, 40, 2030, 2049, 128, True, MSD, "rows", True),
    (2, 8, 2, 5, 4156, 4161, 128, True, MSD, "rows", True),
    (2, 2, 2, 33, 0, 3000, 64, False, MSD, "rows", True),
    (2, 16, 2, 145, 7, 300, 128, True, MSD, "rows", False),
    (2, 16, 2, 129, 140, 257, 64, True, MSD, "rows", False),
    # test_many_rows_d64
    (14, 6, 6, 1000, 0, 1000, 64, False, (P.MIXED, P.DIRECT), "fwd4", False),
    (14, 8, 8, 1100, 0, 1100, 64, True, (P.MIXED, P.DIRECT), "fwd4", False),
    (15, 5, 5, 905, 0, 905, 64, True, (P.MIXED, P.DIRECT), "fwd4", False),
    (14, 8, 8, 900, 350, 1200, 64, True, (P.MIXED, P.DIRECT), "fwd4", False),
    (1, 2, 2, 9000, 0, 9000, 64, True, (P.MIXED, P.DIRECT), "fwd4", True),
    # test_many_rows_d64_in_the_smallest_workspace
    (1, 70, 1, 1000, 0, 1000, 64, False, (P.MIXED,), "fwd4", False),
    (1, 70, 1, 1024, 0, 1024, 64, False, (P.MIXED,), "fwd4", False),
    (1, 70, 1, 1024, 0, 1024, 64, True, (P.MIXED,), "fwd4", False),
    # test_workgroups_of_two_halves
    (1, 28, 4, 1024, 0, 1024, 128, True, MSD, "halves", False),
    (1, 28, 4, 900, 0, 900, 128, False, MSD, "halves", False),
    (1, 28, 4, 1028, 0, 1028, 128, False, MSD, "halves", False),
    (1, 28, 4, 1100, 0, 1100, 128, True, MSD, "halves", False),
    (1, 28, 4, 1000, 900, 2200, 128, True, MSD, "halves", False),
])
def test_calls_reach_the_kernel_they_test(B, Hq, Hkv, Nq, row0, N, d, causal, variants, kernel, split):
    for variant in variants:
        got, nsplit = plan_of(variant, B, Hq, Hkv, Nq, row0, N, d, causal)
        assert got == kernel and (nsplit > 1) == split, (variant, got, nsplit)


@pytest.mark.parametrize("B,Hq,Hkv,N,causal,blocks", [
    (1, 28, 4, 1024, True, 1), (1, 28, 4, 900, False, 1), (1, 28, 4, 1028, False, 2), (1, 28, 4, 1100, True, 1),
    (1, 12, 2, 2304, True, 1), (1, 8, 8, 4000, True, 1), (1, 8, 8, 4000, False, 2), (1, 28, 4, 1500, True, 2), (1, 28, 4, 2048, True, 2),
])
def test_workgroups_of_two_halves_take_the_mfmas_that_were_measured_fastest(B, Hq, Hkv, N, causal, blocks):
    for variant in MSD:
        assert plan_of(variant, B, Hq, Hkv, N, 0, N, 128, causal)[0] == "halves" and row_blocks_of(variant, B, Hq, Hkv, N, 0, N, 128, causal) == blocks


# us of the kernel named / of the one that the estimates once chose, which were fitted to calls of 150 to 6000 keys
@pytest.mark.parametrize("variant,B,Hq,Hkv,Nq,row0,N,d,causal,kernel,split", [
    (P.MIXED, 1, 28, 4, 2100, 0, 2100, 128, True, "halves", False),              # 42.8 / fwd 48.1
    (P.MIXED, 1, 28, 4, 2240, 0, 2240, 128, True, "halves", False),              # 45.6 / fwd 53.9
    (P.MIXED, 1, 28, 4, 841, 0, 841, 128, True, "halves", False),                # 16.7 / rows 20.0
    (P.S16, 1, 32, 8, 1737, 0, 1737, 128, True, "halves", False),                # 36.4 / fwd 48.0
    (P.MIXED, 1, 28, 4, 16640, 0, 16640, 128, False, "fwd", False),              # 3656 / halves 3769
    (P.MIXED, 1, 28, 4, 1391, 0, 10334, 128, False, "fwd", False),               # 216 / halves 273
    (P.S16, 2, 12, 2, 1345, 0, 19387, 128, False, "fwd", False),                 # 435 / halves 560
    (P.S16, 1, 12, 2, 569, 0, 569, 128, False, "rows", False),                   # 11.5 / halves 15.3
    (P.MIXED, 1, 32, 8, 496, 0, 496, 128, False, "rows", False),                 # 11.2 / halves 13.7
    (P.MIXED, 1, 8, 8, 1595, 0, 23274, 128, False, "rows", False),               # 227 / halves 252
    (P.MIXED, 14, 12, 2, 5, 0, 2301, 128, False, "rows", True),                  # 12.7 / in one piece 15.2
    (P.MIXED, 1, 1, 1, 6042, 0, 6042, 64, True, "rows", True),                   # 20.2 / in one piece 26.8
    (P.MIXED, 2, 1, 1, 28830, 0, 28830, 64, True, "fwd4", False),                # 354 / rows 558
    (P.MIXED, 4, 1, 1, 12590, 0, 12590, 64, True, "fwd4", False),                # 154 / rows 176
    (P.MIXED, 14, 16, 16, 186, 7820, 8006, 64, True, "fwd", False),              # 148 / fwd4 166
])
def test_calls_go_to_the_kernel_that_was_measured_fastest(variant, B, Hq, Hkv, Nq, row0, N, d, causal, kernel, split):
    got, nsplit = plan_of(variant, B, Hq, Hkv, Nq, row0, N, d, causal)
    assert got == kernel and (nsplit > 1) == split, (got, nsplit)


def test_what_the_workspace_holds_cuts_the_pieces():
    """Two pieces are not asked for where the rows of a KV head are one block, but may be all that the split region holds."""
    assert plan_of(P.MIXED, 24, 8, 8, 1, 3999, 4000, 128, True) == ("rows", 1)             # 192 workgroups: not two
    assert plan_of(P.MIXED, 28, 28, 4, 1, 4999, 5000, 128, True) == ("rows", 2)            # 112 workgroups: four wanted
    bare = P.pasa_attn_fwd_workspace_min(28, 4, 5000, 128)
    assert plan_of(P.MIXED, 28, 28, 4, 1, 4999, 5000, 128, True, workspace_bytes=bare) == ("rows", 1)
    assert plan_of(P.MIXED, 28, 28, 4, 1, 4999, 5000, 128, True, workspace_bytes=bare + (4 << 20)) == ("rows", 4)


def test_pieces_are_planned_as_the_whole():
    """Wherever a whole sequence's keys are swept unsplit, its pieces of 32 rows or more go to its kernel, and unsplit."""
    import random
    rng, pieces = random.Random(4), 0
    while pieces < 5000:
        B, (Hq, Hkv, d) = rng.choice([1, 1, 2, 4, 14]), rng.choice([(28, 4, 128), (8, 8, 128), (12, 2, 128), (2, 2, 128), (5, 5, 64), (16, 16, 64), (1, 1, 64)])
        N, causal, variant = int(2 ** rng.uniform(5, 15)), rng.random() < 0.6, rng.choice([P.MIXED, P.DIRECT, P.S16])
        Nq = rng.randint(32, min(N, 4096))
        if N > 2048 and -(-Nq // 256) * Hq * B < 192:
            continue
        row0 = rng.randint(0, (N - Nq) // 32) * 32 if causal else 0
        whole, piece = (plan_of(variant, B, Hq, Hkv, n, r, N, d, causal) for n, r in ((N, 0), (Nq, row0)))
        assert piece == (whole[0], 1), (variant, B, Hq, Hkv, Nq, row0, N, d, causal, whole, piece)
        pieces += 1


def test_counters_and_fp16_state_stay_on_the_256_row_kernel():
    for variant in (P.MIXED, P.S16, P.DIRECT, P.STRICT16, P.NAIVE16):
        for N in (1, 300, 1024, 9000):
            for d in (64, 128):
                assert plan_of(variant, 1, 28, 4, N, 0, N, d, True, counters=True)[0] == "fwd"
                if variant in (P.STRICT16, P.NAIVE16):
                    assert plan_of(variant, 1, 28, 4, N, 0, N, d, True)[0] == "fwd"


def test_division_by_a_number_that_the_host_knows():
    """Exact for every n below 2^31: multiples of the divisor and their neighbours are where a rounded reciprocal goes wrong."""
    import ctypes
    import random
    import torch  # noqa: F401  before the library, which then shares the HIP runtime that torch brings
    f = P.lib().pasa_internal_quotient
    f.argtypes, f.restype = [ctypes.c_uint, ctypes.c_uint], ctypes.c_uint
    rng = random.Random(3)
    top = (1 << 31) - 1
    for d in [1, 2, 3, 5, 7, 28, 64, 65, 641, 262143, 262144, 6700417, (1 << 30) - 1, 1 << 30, (1 << 30) + 1, top] + [rng.randint(1, top) for _ in range(300)]:
        for q in [0, 1, 2, top // d - 1, top // d] + [rng.randint(0, top // d) for _ in range(20)]:
            for n in (q * d - 1, q * d, q * d + 1, top):
                if 0 <= n <= top:
                    assert f(n, d) == n // d, (n, d)
