"""The host's plans for the team kernel against the dealing rule of the kernel, on the CPU: for every number of row blocks that the
device may form, every stage of every column block belongs to one sum, the sums of a block lie in planes 0, 1, ... below the number
the consumer sums, and none is longer than the limit."""
import ctypes as C

import pytest

from paper_2410_13344_amd import binding as B

STAGE_COLUMNS = 64          # columns of K per stage
BLOCK_COLUMNS = 512         # columns of a column block


class Plan(C.Structure):
    _fields_ = [("NT", C.c_int), ("planes", C.c_int), ("grid", C.c_int), ("rb_min", C.c_int), ("t_max", C.c_int), ("chain", C.c_int),
                ("planes_of", C.c_ulonglong * 2), ("RB", C.c_int), ("rows_per", C.c_int), ("T", C.c_int)]


def plan(rows_max, N, K, cus, max_planes, live, k_chain):
    f = getattr(B.lib(), "_ZN4cerb14plan_team_gemmEiiiiibiPNS_8TeamPlanE")     # bool plan_team_gemm(int x 5, bool, int, TeamPlan*)
    f.restype, f.argtypes = C.c_bool, [C.c_int] * 5 + [C.c_bool, C.c_int, C.POINTER(Plan)]
    p = Plan()
    return p if f(rows_max, N, K, cus, max_planes, live, k_chain, C.byref(p)) else None


def sums(stages, chain):
    """Lengths of the sums that a team's stages of a column block are cut into."""
    if chain <= 0 or stages <= chain:
        return [stages]
    n = -(-stages // chain)
    each = -(-stages // n)
    return [min(each, stages - i) for i in range(0, stages, each)]


def check(p, rows_max, N, K, cus, live):
    nst, blocks = K // STAGE_COLUMNS, -(-(N // 16) // (BLOCK_COLUMNS // 16))
    units = blocks * nst
    assert 5 <= p.NT <= 8 and p.grid == cus
    for RB in range(p.rb_min, max(p.rb_min, -(-rows_max // (16 * p.NT))) + 1):
        T = min(cus // RB, p.t_max, units)
        assert T >= 1
        planes = (p.planes_of[RB >> 4] >> ((RB & 15) * 4) & 15) + 1 if live else p.planes
        assert planes <= p.planes
        covered, used = 0, [0] * blocks
        for t in range(T):
            v, v1 = units * t // T, units * (t + 1) // T
            while v < v1:
                cb = v // nst
                stop = min(v1, (cb + 1) * nst)
                lengths = sums(stop - v, p.chain)
                assert sum(lengths) == stop - v and min(lengths) > 0 and (p.chain <= 0 or max(lengths) <= p.chain)
                used[cb] += len(lengths)
                covered += stop - v
                v = stop
        assert covered == units and max(used) <= planes, (RB, T, max(used), planes)
        if live:
            assert max(used) == planes


SHAPES = [(4096, 11008), (5120, 13824), (12288, 4096), (15360, 5120), (22016, 4096), (27648, 5120), (32000, 4096), (1024, 1024), (3072, 1024),
          (768, 256), (2000, 256), (2048, 1024), (8192, 28672), (65536, 8192), (16, 256)]


@pytest.mark.parametrize("N,K", SHAPES)
def test_plans_cover_every_shape_that_the_device_may_take(N, K):
    made = 0
    for rows_max in list(range(129, 640, 37)) + [768, 769, 896, 968, 1024, 1025, 1152, 1936, 2048, 3071, 3072]:
        for max_planes in (1, 4, 8, 16):
            plain = plan(rows_max, N, K, 256, max_planes, False, 0)
            live = plan(rows_max, N, K, 256, max_planes, True, 0)
            assert (plain is None) == (live is None)            # the same launches take the kernel either way
            for p, is_live in ((plain, False), (live, True)):
                if p:
                    made += 1
                    assert p.planes <= max_planes and p.chain == 0
                    check(p, rows_max, N, K, 256, is_live)
            if plain:
                assert live.rb_min <= plain.rb_min and (live.RB, live.rows_per) == (plain.RB, plain.rows_per)
            for splits in (2, 3, 8):                            # as long as the longest of so many ranges of K
                k_chain = -(-(K // 128) // splits) * 128
                p = plan(rows_max, N, K, 256, max_planes, False, k_chain)
                if p:
                    made += 1
                    assert p.planes <= max_planes and p.chain == k_chain // STAGE_COLUMNS
                    check(p, rows_max, N, K, 256, False)
    assert made > 0


def test_shapes_that_the_kernel_does_not_take():
    assert plan(128, 4096, 4096, 256, 8, False, 0) is None
    assert plan(1024, 4100, 4096, 256, 8, True, 0) is None
    assert plan(1024, 4096, 4096 + 32, 256, 8, True, 0) is None
    assert plan(1024, 4096, 4096, 4, 8, True, 0) is None
    assert plan(1024, 4096, 11008, 256, 8, True, 0).planes == 8 and plan(1024, 4096, 11008, 256, 8, False, 0).planes == 5
