"""The rules that choose between forms of a kernel (csrc/rules.h), at shapes where both forms were timed:
the faster one has to be chosen wherever they differ by more than 5%."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "rules")
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_1912_00539_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host", "rules.cpp"), "-o", exe])

    def ask(rule, *args):
        rc = subprocess.run([exe, rule] + [str(int(a)) for a in args]).returncode
        assert rc in (0, 1), (rule, rc)
        return rc == 1
    return ask


# cells, rows per chunk, blocks a side, FP64, time of three sweeps each way: a quad, sixteen lanes per chunk
CHAIN_APPLY = [(500000, 1, 2, 0, 177, 563), (500000, 2, 2, 0, 167, 287), (500000, 3, 2, 0, 158, 205),
               (500000, 5, 2, 0, 177, 146), (500000, 16, 2, 0, 156, 112), (500000, 1, 2, 1, 279, 1153),
               (500000, 4, 2, 1, 270, 338), (500000, 10, 2, 1, 285, 228), (500000, 64, 2, 1, 598, 223),
               (500000, 4, 3, 0, 200, 240), (500000, 6, 3, 0, 221, 194), (500000, 8, 3, 1, 345, 408),
               (500000, 12, 3, 1, 394, 345), (120000, 4, 2, 0, 47, 56), (120000, 6, 2, 0, 54, 45),
               (120000, 6, 2, 1, 77, 82), (120000, 8, 2, 1, 84, 75), (10057, 1, 2, 0, 25, 32), (10057, 3, 2, 0, 30, 26),
               (10057, 2, 2, 1, 30, 35), (10057, 3, 2, 1, 33, 27), (64000, 3, 3, 0, 42, 55), (64000, 5, 3, 0, 48, 44),
               (64000, 5, 3, 1, 68, 86), (64000, 8, 3, 1, 84, 56)]


@pytest.mark.parametrize("n,R,side,f64,quad,sixteen", CHAIN_APPLY)
def test_chain_apply(rules, n, R, side, f64, quad, sixteen):
    assert rules("chain_apply", R, -(-n // R), side, f64) == (sixteen < quad)


# cells, rows per chunk, blocks a side, FP64, from A, time of a sweep: whole rows, two launches
CHAIN_FACTOR = [(500000, 1, 2, 0, 1, 124, 173), (500000, 2, 2, 0, 1, 152, 160), (500000, 8, 2, 0, 1, 164, 158),
                (500000, 6, 2, 0, 1, 167, 157), (120000, 6, 2, 0, 1, 39, 42),
                (500000, 64, 2, 0, 1, 239, 183), (120000, 1, 2, 0, 1, 34, 47), (120000, 16, 2, 0, 1, 57, 46),
                (10057, 4, 2, 0, 1, 15, 13), (10057, 16, 2, 0, 1, 44, 24), (500000, 1, 2, 0, 0, 195, 261),
                (500000, 4, 2, 0, 0, 231, 254), (500000, 16, 2, 0, 0, 241, 259), (500000, 64, 2, 0, 0, 293, 275),
                (500000, 128, 2, 0, 0, 461, 327), (120000, 4, 2, 0, 0, 47, 54), (120000, 16, 2, 0, 0, 67, 60),
                (10057, 1, 2, 0, 0, 14, 18), (10057, 3, 2, 0, 0, 16, 18), (10057, 8, 2, 0, 0, 28, 21),
                (500000, 1, 2, 1, 1, 233, 208), (500000, 16, 2, 1, 1, 250, 211), (10057, 1, 2, 1, 0, 17, 19),
                (10057, 4, 2, 1, 0, 28, 23), (500000, 64, 2, 1, 0, 547, 420), (500000, 1, 3, 0, 0, 313, 329),
                (500000, 5, 3, 0, 0, 370, 324), (64000, 1, 3, 1, 1, 44, 38), (64000, 3, 3, 0, 1, 34, 30)]


@pytest.mark.parametrize("n,R,side,f64,from_a,whole,two", CHAIN_FACTOR)
def test_chain_factor(rules, n, R, side, f64, from_a, whole, two):
    assert rules("chain_factor", R, -(-n // R), side, f64, from_a) == (two < whole)


# cells, lower blocks, blocks a side, farthest neighbour, FP64, time of three sweeps each way: single, pairs
SWEEP_PAIRS = [(64000, 187200, 3, 1600, 0, 21.7, 16.4), (72000, 200000, 3, 14400, 0, 22.7, 21.3),
               (700000, 2062000, 3, 400, 0, 156, 149), (700700, 2085000, 3, 4900, 0, 158, 166),
               (700000, 2079000, 3, 10000, 0, 160, 177), (720000, 2140000, 3, 14400, 0, 161, 186),
               (700000, 2062000, 3, 400, 1, 284, 230), (720000, 2140000, 3, 14400, 1, 298, 276),
               (600000, 900000, 3, 3000, 0, 108, 80), (700000, 1400000, 2, 4000, 0, 113, 95),
               (700000, 1400000, 2, 12000, 0, 114, 107), (700000, 1400000, 2, 12000, 1, 208, 175),
               (180000, 270000, 3, 180000, 0, 39.6, 54.5), (800000, 1200000, 3, 800000, 1, 246, 321)]


@pytest.mark.parametrize("n,ZL,side,far,f64,single,pairs", SWEEP_PAIRS)
def test_sweep_pairs(rules, n, ZL, side, far, f64, single, pairs):
    args = side, far <= 16384, far <= 2048, n, ZL, f64
    assert rules("sweep_pairs", 3, *args) == (pairs < single)
    assert not rules("sweep_pairs", 2, *args) and not rules("sweep_pairs", 3, 4, *args[1:])


# cells, blocks, time of an asynchronous FP64 sweep from A: as many workgroups as fit, three a compute unit
CROWDED_SWEEP = [(57600, 1460000, 346, 418), (100000, 2600000, 642, 558), (180000, 4700000, 1133, 997),
                 (294000, 7700000, 1885, 1602), (560000, 3900000, 385, 432), (700000, 4800000, 400, 442)]


@pytest.mark.parametrize("n,Z,fit,three", CROWDED_SWEEP)
def test_crowded_sweep(rules, n, Z, fit, three):
    assert rules("crowded_sweep", n, Z) == (three < fit)


# cells, blocks, neighbours near, FP64, from A, time of a synchronous sweep: a quad per row, per block
SWEEP_BY_BLOCKS = [(400000, 2760000, 0, 0, 1, 152, 141), (550000, 3810000, 0, 0, 1, 240, 254),
                   (700000, 4840000, 0, 0, 1, 306, 335), (800000, 3996000, 0, 0, 1, 251, 265),
                   (800000, 3996000, 1, 0, 1, 228, 162), (700000, 4840000, 0, 1, 1, 474, 428),
                   (150000, 1030000, 0, 1, 1, 90, 78), (249900, 1720000, 0, 1, 0, 253, 260),
                   (700000, 4840000, 0, 1, 0, 679, 722), (800000, 3996000, 0, 1, 0, 571, 604),
                   (90000, 448800, 0, 1, 0, 60, 58), (800000, 3996000, 1, 1, 0, 554, 548),
                   (249900, 1720000, 0, 0, 0, 165, 160)]


@pytest.mark.parametrize("n,Z,near,f64,from_a,row,block", SWEEP_BY_BLOCKS)
def test_sweep_by_blocks(rules, n, Z, near, f64, from_a, row, block):
    ZL = (Z - n) // 2
    assert rules("sweep_by_blocks", n, Z, ZL, ZL, near, f64, from_a) == (block < row)
    assert rules("sweep_by_blocks", n, Z, ZL, ZL + 1, near, f64, from_a)   # update sets off the diagonal


# rows, blocks, times of a solve to 1e-10 and of one of two iterations or one: none, one, two launches ahead
AHEAD = [(9940, 39478, 298, 295, 286), (48000, 191380, 406.3, 404.3, 373.2), (48000, 191380, 164.9, 157.2, 151.6),
         (180000, 718800, 716, 678, 689), (121797, 850353, 616, 590, 595), (250000, 1248000, 923, 896, 920),
         (700000, 2797600, 591, 621, 666), (180000, 4689232, 1454, 1468, 1509), (180000, 4689232, 499, 529, 570),
         (40000, 199120, 437.5, 428.0, 418.5), (60000, 298900, 492.7, 476.5, 465.1), (24000, 168000, 571.9, 537.1, 526.2),
         (24000, 168000, 182.4, 176.8, 176.3), (230000, 1600000, 1875.5, 1829.3, 1838.7),
         (400000, 2800000, 2971.1, 2906.5, 2944.3), (400000, 2800000, 921.8, 930.6, 959.1),
         (8000, 195112, 216.6, 212.8, 220.2), (57600, 1475944, 849.3, 839.0, 849.2), (57600, 1475944, 208, 207, 219)]


@pytest.mark.parametrize("rows,blocks,none,one,two", AHEAD)
def test_launches_ahead(rules, rows, blocks, none, one, two):
    """Within the 2% by which runs of one side differ of the best."""
    taken = [k for k in range(3) if rules("launches_ahead", rows, blocks, k)]
    assert len(taken) == 1 and (none, one, two)[taken[0]] <= 1.02 * min(none, one, two)


@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("nsw", [0, 1, 2, 3, 4, 5, 6, 7, 8])
def test_direction_of_the_last_backward_launch(rules, nsw, pairs):
    """The launches as the application makes them: the first descending, then in turn."""
    q, desc = 2, []
    while q <= nsw:
        desc.append(len(desc) % 2 == 0)
        assert rules("backward_descends", len(desc) - 1) == desc[-1]
        q += 2 if pairs and q + 1 <= nsw else 1
    assert rules("apply_ends_descending", nsw, pairs) == (bool(desc) and desc[-1])
