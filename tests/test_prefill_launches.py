"""CPU: the matrix launches of a grouped prefill call (csrc/lcd_gemm_plan.h): wide and split layers share a launch only with tiles that the kernel for
both has, and tiles that are launched apart are the best of their own."""
import random

from gemm_plan import HALVES, SPLIT, choices, launches


def _groups():
    rng = random.Random(3)
    for _ in range(3000):
        K = 256 * rng.randint(1, 44)
        yield rng.choice([2, 3, 4]), int(2 ** rng.uniform(5, 11.5)), [(16 * int(2 ** rng.uniform(4, 10)), K if rng.random() < 0.7 else 256 * rng.randint(1, 44)) for _ in range(rng.randint(2, 5))]


def test_launches_of_wide_and_split_layers():
    cases = list(_groups())
    plans = launches(cases)
    wide = [(b, M, [l for l, k in zip(ls, kernels) if k == HALVES]) for (b, M, ls), (kernels, *_) in zip(cases, plans)]
    alone = iter(choices([(0, b, M, ls) for b, M, ls in wide if ls]))
    seen = {True: 0, False: 0}
    for (bits, M, layers), (kernels, together, halves, split), (_, _, wide_layers) in zip(cases, plans, wide):
        assert (halves[3] > 0) == (HALVES in kernels) and (split[0] > 0) == (SPLIT in kernels)
        best = next(alone) if wide_layers else None
        if together:
            assert HALVES in kernels and SPLIT in kernels
            form, blocks, big, columns = halves
            assert form in (0, 1) and (blocks == 4 or (blocks == 3 and big == columns))
            assert big * blocks + (columns - big) * (blocks - 1) == -(-M // 32)
            assert split in ((2, 3), (2, 4))
        elif HALVES in kernels:
            assert halves == best
        if HALVES in kernels and SPLIT in kernels:
            seen[together] += 1
    assert seen[True] > 300 and seen[False] > 10, seen


def test_grouped_query_attention_is_one_launch():
    for kv, shapes, M in ((1280, (5120, 5120), 500), (1024, (4096, 4096), 700), (1024, (8192, 8192), 333)):
        for bits in (2, 3, 4):
            kernels, together, *_ = launches([(bits, M, [shapes, (kv, shapes[1]), (kv, shapes[1])])])[0]
            assert kernels == (HALVES, SPLIT, SPLIT) and together, (bits, shapes)
