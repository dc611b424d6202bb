"""The tiled GEMM's choice of tile and K split, on the CPU: partial tiles fit the scratch they are given whatever the
shape (a single split's too), only tiles that exist for the type and epilogue are chosen, what is not
partial tiles is not split, and shapes the kernel does not take get no plan."""
import ctypes as C
import random

from paper_2502_09922_amd import binding

F32, BF16 = 0, 1
PART, STORE, SWIGLU, ROPE = range(4)


class Plan:
    def __init__(self, bm, bn, splits):
        self.bm, self.bn, self.splits = bm, bn, splits


def plan(dt, epi, m, n, k, to_scratch, scratch):
    fn = binding.lib.ls_test_tiled_plan
    fn.argtypes = [C.c_uint32, C.c_int, C.c_int, C.c_int, C.c_int, C.c_int, C.c_size_t, C.POINTER(C.c_int * 3)]
    out = (C.c_int * 3)()
    fn(dt, epi, m, n, k, to_scratch, scratch, C.byref(out))
    return Plan(*out)


def test_plans_over_random_shapes():
    rng = random.Random(7)
    seen = set()
    for _ in range(20000):
        dt, epi = rng.choice([F32, BF16]), rng.choice([PART, STORE, SWIGLU, ROPE])
        m = int(2 ** rng.uniform(0, 15))
        n, k = 16 * rng.randint(1, 1800), rng.choice([16, 32, 128]) * rng.randint(1, 220)
        scratch = rng.choice([0, 1 << 16, 16 << 20, 64 << 20])
        p = plan(dt, epi, m, n, k, epi == PART, scratch)
        if not p.splits:
            continue
        if epi == PART:
            assert p.splits * m * n * 4 <= scratch, (dt, m, n, k, scratch, p.splits)
        else:
            assert p.splits == 1
        if p.bm == 0:
            assert dt == F32 and m <= 8 and epi != ROPE and k % 4 == 0
            continue
        assert k % (16 if dt == F32 else 32) == 0 and k >= 64
        assert not (dt == F32 and p.bn == 256) and not (epi == SWIGLU and p.bn == 64)
        assert p.splits == 1 or -(-k // (32 if dt == F32 else 64)) >= 2 * p.splits  # k-steps of a split
        seen.add((dt, p.bm, p.bn))
    assert len(seen) >= 14  # the rule spreads over the tiles there are


def test_no_plan_for_what_the_kernel_does_not_take():
    big = 64 << 20
    for dt, m, n, k in ((BF16, 40, 100, 512), (BF16, 40, 512, 48), (F32, 40, 512, 72), (F32, 40, 8, 64), (BF16, 40, 1 << 20, 1 << 14)):
        assert plan(dt, STORE, m, n, k, False, 0).splits == 0
    assert plan(BF16, PART, 3000, 8192, 8192, True, big).splits == 0  # 98 MB of partial tiles
    assert plan(BF16, PART, 2000, 8192, 8192, True, big).splits == 1


def test_launches_with_a_chosen_tile_that_are_refused():
    """Nothing is launched for what the kernels do not take: other tiles, K not of half k-steps, a cut matrix that is not
    partial tiles, more parts than K has, SwiGLU where gate and up do not lie in one wavefront."""
    fn = binding.lib.ls_test_tiled_gemm
    fn.argtypes = [C.c_uint32] + [C.c_int] * 4 + [C.c_void_p] * 2 + [C.c_int] * 3 + [C.c_void_p] * 2
    p = 256  # never read
    for dt, epi, bm, bn, splits, m, n, k in ((F32, STORE, 160, 256, 1, 40, 64, 64), (BF16, STORE, 48, 128, 1, 40, 64, 64),
                                             (F32, STORE, 160, 128, 1, 40, 64, 64), (F32, STORE, 256, 128, 1, 40, 64, 64),
                                             (F32, STORE, 0, 0, 1, 4, 64, 64), (BF16, STORE, 32, 64, 1, 40, 64, 80),
                                             (F32, STORE, 32, 64, 2, 40, 64, 512), (F32, PART, 32, 64, 5, 40, 64, 256),
                                             (BF16, SWIGLU, 64, 64, 1, 40, 64, 64), (BF16, STORE, 32, 64, 1, 40, 24, 64),
                                             (F32, ROPE, 32, 64, 1, 40, 64, 64)):
        assert not fn(dt, epi, bm, bn, splits, p, p, m, n, k, p, None)


def test_fp32_by_split_operands_only_where_it_pays():
    """The kernel that splits the rows in front and the tall tiles cost small matrices more than they save (512 columns, 97..512
    rows: 175..263 us for two layers against 103..196); at the 7B shape they are the faster ones from some 70 rows on."""
    for d, f in ((256, 688), (384, 1024), (512, 1376)):
        for m in (97, 128, 200, 311, 512):
            for epi, n, k in ((ROPE, 3 * d, d), (PART, d, d), (SWIGLU, f, d), (PART, d, f)):
                p = plan(F32, epi, m, n, k, epi == PART, 8 * m * n * 4)
                assert p.bm * p.bn < 96 * 128, (d, m, epi, p.bm, p.bn)
    assert [(p.bm, p.bn) for p in (plan(F32, SWIGLU, m, 688, 256, False, 0) for m in (97, 200, 512))] == [(32, 128)] * 3
    for m in (97, 200, 325, 1000):
        for epi, n, k in ((ROPE, 12288, 4096), (PART, 4096, 4096), (SWIGLU, 11008, 4096), (PART, 4096, 11008)):
            p = plan(F32, epi, m, n, k, epi == PART, 64 << 20)
            assert p.bm * p.bn >= 96 * 128, (m, epi, p.bm, p.bn)


def test_one_tile_row_before_two_of_the_same_lines():
    """Gate-up of 7B, 121..136 rows, and of 13B and 70B, 249..256 rows: measured 7 to 10 % faster in one tile row."""
    for m in (121, 124, 128):
        assert (plan(BF16, SWIGLU, m, 11008, 4096, False, 0).bm, plan(BF16, SWIGLU, m, 11008, 4096, False, 0).bn) == (128, 128)
    for m in (249, 256):
        for n, k in ((13824, 5120), (28672, 8192)):
            assert (plan(BF16, SWIGLU, m, n, k, False, 0).bm, plan(BF16, SWIGLU, m, n, k, False, 0).bn) == (256, 128)
