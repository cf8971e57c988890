"""Rules of the GEMM planner (csrc/gemm_plan.hpp), compiled with a host compiler: no GPU involved."""
import os
import subprocess

import pytest

from paper_2507_06608_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHARES = range(32, 257, 32)
MODELS = ("llama3_8b", "qwen25_14b", "llama3_70b")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "gemm_plan")
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-o", exe, os.path.join(ROOT, "tests", "gemm_plan_driver.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def run(lines):
        r = subprocess.run([exe], input="".join(l + "\n" for l in lines), capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        out = [tuple(int(x) for x in l.split()) for l in r.stdout.splitlines()]
        assert len(out) == len(lines)
        return out
    return run


def projections(s):
    """(features, K, own reduction) of a layer's four projections."""
    return [(s.n_qkv, s.hidden, 0), (s.hidden, s.q_dim, 0), (2 * s.ffn, s.hidden, 1), (s.hidden, s.ffn, 0)]


@pytest.mark.parametrize("shape", MODELS)
def test_slices_up_to_128_rows_suit_every_share(ask, shape):
    """The number of K slices cannot follow the CU share (it is the order of summation), so it has to suit all of them: the CU that
    loads most loads at most 1.8 times its part of a split projection (2 slots of a CU for w workgroups on c CUs are 2 c / w times; the
    grids of these shapes reach 1.75, and 240 workgroups, which suit 256 CUs best, are 1.87 on 224 and up to 8 % of a step)."""
    projs = projections(synth.SHAPES[shape])
    rows = [1, 23, 32, 33, 64, 65, 128]
    plans = ask([f"plan {t} {n // 32} {k} {own}" for t in rows for n, k, own in projs])
    for i, (s, _, fs, ts) in enumerate(plans):
        n, t = projs[i % 4][0], rows[i // 4]
        blocks = -(-(n // 32) // fs) * -(-(-(-t // 32)) // ts)
        assert s == 1 or blocks * s >= 192 or s == 8, (t, n, s)
        for c in SHARES:
            if s > 1:
                assert -(-blocks * s // c) * c <= 1.8 * blocks * s, (t, n, s, c)


# tiles, blocks of tokens, slices, CUs of the share, dealt in ranges?  Of the grids whose kernels were timed in both orders.
ORDERS = [(180, 2, 1, 192, True), (174, 2, 1, 176, True), (180, 2, 1, 208, True), (44, 2, 4, 176, True), (86, 2, 2, 176, True),  # faster in ranges
          (180, 2, 1, 176, False), (300, 2, 1, 160, False), (44, 2, 4, 168, False),              # more than one round
          (86, 2, 1, 96, False), (44, 2, 2, 96, False), (46, 2, 2, 128, False),                  # half of the chip and less
          (270, 3, 1, 160, False), (135, 5, 1, 192, False), (540, 3, 1, 192, False), (52, 4, 4, 224, False),  # three and more blocks of tokens
          (180, 2, 1, 256, False), (22, 1, 4, 96, False), (150, 1, 1, 160, False),               # the whole chip; one block
          (176, 2, 1, 192, True), (256, 3, 2, 256, True), (8, 1, 1, 64, True)]                   # multiples of the XCDs


@pytest.mark.parametrize("tiles,n_tblk,slices,cus,ranges", ORDERS, ids=[f"{o[0]} tiles, {o[1]} blocks, {o[2]} slices, {o[3]} CUs" for o in ORDERS])
def test_which_grids_are_dealt_in_ranges(ask, tiles, n_tblk, slices, cus, ranges):
    assert ask([f"xcds {tiles} {n_tblk} {slices} {cus}"]) == [(8 if ranges else 1,)]


def test_every_tile_is_computed_once(ask):
    """tile_of_block, which the kernel calls, is a permutation of the tiles for any grid and number of XCDs, and an XCD's workgroups
    (they are dealt round-robin) hold one contiguous range of tiles."""
    grids = [(n, x) for x in (1, 2, 7, 8) for n in list(range(1, 600)) + [4096, 4099]]
    for (n, x), order in zip(grids, ask([f"order {n} {x} 0 0" for n, x in grids])):
        assert sorted(order) == list(range(n)), (n, x)
        for d in range(x):
            mine = order[d::x]
            assert x == 1 or list(mine) == list(range(mine[0], mine[0] + len(mine))) if mine else True, (n, x, d)
