"""Which kernel a matrix product runs on: the rules of csrc/gemm_plan.h, evaluated on
the CPU."""

from __future__ import annotations

import collections
import csv
import os
import shutil
import subprocess

import numpy as np
import pytest

from tests.test_gpu_rows import CFGS, TILE_CFGS, TILE_ROWS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GXX = shutil.which("g++")
BF16, Q8 = 1, 2

pytestmark = pytest.mark.skipif(GXX is None, reason="g++ not available")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """Answers (tuples of ints) to a list of questions (see the harness)."""
    exe = str(tmp_path_factory.mktemp("plan") / "plan")
    subprocess.run([GXX, "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2608_24204_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "plan_harness.cpp"), "-o", exe], check=True)

    def run(questions):
        text = "".join(" ".join(map(str, q)) + "\n" for q in questions)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60)
        out = [tuple(map(int, l.split())) for l in r.stdout.splitlines()]
        assert len(out) == len(questions)
        return out

    return run


def test_ranges_are_whole_and_the_launch_agrees(ask):
    """Over random shapes: K ranges of whole steps, no more than asked for, and a launch
    that is given the count picks the kernel that the count was made for."""
    rng = np.random.default_rng(0)
    qs = []
    for _ in range(20000):
        wt, nt = int(rng.choice([BF16, Q8])), int(rng.integers(1, 4))
        M = int(np.exp(rng.uniform(0, np.log(8192))))
        N = 64 * int(np.exp(rng.uniform(0, np.log(900)))) + int(rng.choice([0, 0, 1, 37]))
        K = 64 * int(np.exp(rng.uniform(0, np.log(512))))
        qs.append(("ranges", wt, nt, M, N, K, int(rng.integers(1, 9))))
    for q, (n, rows, rows_n) in zip(qs, ask(qs)):
        _, wt, nt, M, N, K, most = q
        assert 1 <= n <= most, q
        assert rows == rows_n, q
        if n > 1:
            assert K % (n * (128 if rows else 64)) == 0, q
    split = [(q, n) for q, (n, rows, _) in zip(qs, ask(qs)) if rows]
    got = ask([("rows",) + q[1:6] + (n,) for q, n in split])
    assert all(p[2] == n for p, (_, n) in zip(got, split))


@pytest.mark.parametrize("M,N,K,most,rows", [
    (64, 4096, 4096, 8, True), (96, 4096, 14336, 8, True), (96, 6144, 4096, 4, True),
    (96, 28672, 4096, 1, True), (128, 28672, 4096, 1, True), (96, 5120, 27648, 8, True),
    (128, 4096, 4096, 8, False), (128, 6144, 4096, 4, False), (96, 2048, 8192, 8, False),
    (96, 55296, 5120, 1, False), (128, 55296, 5120, 1, False), (129, 28672, 4096, 1, False)])
def test_prompts_leave_the_few_row_kernel_where_tiles_are_faster(ask, M, N, K, most, rows):
    """Either side of the lines whose measured times stand beside the rule."""
    assert ask([("ranges", BF16, 2, M, N, K, most)])[0][1] == rows


@pytest.mark.parametrize("M,N,K,rows", [
    (64, 128256, 4096, True), (65, 128256, 4096, False), (128, 152064, 5120, False),
    (80, 55296, 5120, False), (128, 28672, 4096, True), (80, 16384, 2048, False),
    (128, 6144, 4096, True), (128, 3072, 2048, True), (129, 6144, 4096, False)])
def test_batches_leave_the_few_row_kernel_where_tiles_are_faster(ask, M, N, K, rows):
    assert ask([("merge", BF16, 3, M, N, K, 0)])[0][0] == rows


TILES = ["128x256", "128x128", "64x128"]


@pytest.fixture(scope="module")
def measured():
    with open(os.path.join(ROOT, "profiles", "tile_times.csv")) as f:
        return [(r["epilogue"] == "swiglu", TILES.index(r["tile"]), int(r["terms"]), int(r["M"]),
                 int(r["N"]), int(r["K"]), int(r["ranges"]), float(r["us"])) for r in csv.DictReader(f)]


def kind(swiglu):
    return "tileg" if swiglu else "tile"


def test_tiles_that_fit_a_cu(ask):
    """The time model counts as resident the workgroups that the 160 KiB of LDS hold:
    64 bytes a row, activation term and stage, two stages (three of the 64-row tile)."""
    for what in ("fit", "fitg"):
        for nt in (1, 2, 3):
            got = ask([(what, BF16, nt, 0, 0, 0, 0)])[0]
            for s, (bm, bn, fit) in enumerate(zip(got[::3], got[1::3], got[2::3])):
                lds = 64 * (nt * bm + bn) * (3 if TILES[s] == "64x128" else 2)
                assert fit * lds <= 160 * 1024, (TILES[s], nt, fit)


def test_time_model_fits_the_measured_products(ask, measured):
    """As the comment beside the constants says: 8% rms, for each kind of tile and number
    of terms within 10%."""
    got = ask([(kind(g), BF16, nt, M, N, K, n) for g, _, nt, M, N, K, n, _ in measured])
    err = collections.defaultdict(list)
    for (g, s, nt, *_, us), t in zip(measured, got):
        err[s, g and s == 2, nt].append(np.log(t[1 + s] * 1e-3 / us))
    assert np.sqrt(np.mean(np.square(np.concatenate(list(err.values()))))) <= 0.085
    for k, e in err.items():
        assert np.sqrt(np.mean(np.square(e))) <= 0.10, (k, np.sqrt(np.mean(np.square(e))))


def test_chosen_tiles_and_ranges_are_near_the_best_measured(ask, measured):
    """Over the measured products with every tile and count: the chosen pair against the
    fastest one (partials read by the next kernel counted at 0.7 us a million)."""
    by = collections.defaultdict(dict)
    for g, s, nt, M, N, K, n, us in measured:
        by[g, nt, M, N, K][n, s] = us + (0.7e-6 * n * M * N if n > 1 else 0.0)
    keys, most = [], {}
    for k, d in by.items():
        if k[0] or k[2] > 128:                 # fewer rows: the few-row kernel's
            keys.append(k)
            most[k] = 1 if k[0] else 8
    ranges = [r[0] for r in ask([("ranges", BF16, k[1], k[2], k[3], k[4], most[k]) for k in keys])]
    shapes = [t[0] for t in ask([(kind(k[0]), BF16, *k[1:], n) for k, n in zip(keys, ranges)])]
    loss = []
    for k, n, s in zip(keys, ranges, shapes):
        if (n, s) in by[k]:                    # counts of 3, 5, 6, 7 are measured for some only
            loss.append(by[k][n, s] / min(by[k].values()))
    assert len(loss) > 0.9 * len(keys)
    assert np.mean(loss) <= 1.045 and np.max(loss) <= 1.40, (np.mean(loss), np.max(loss))


def prompt_products(ask, cfg, M, chunk=2048):
    """(kernel, ranges, N, K) of the four products of a prompt of M rows: the rules as the
    prefill applies them, with the default mode's activation terms (3, 2, 2, 2)."""
    d, F, qd = cfg.d_model, cfg.ffn_dim, cfg.n_heads * cfg.head_dim
    out = {}
    for name, nt, N, K, most in (("qkv", 3, qd + 2 * cfg.n_kv_heads * cfg.head_dim, d, 4),
                                 ("o", 2, d, qd, 8), ("gu", 2, 2 * F, d, 1), ("down", 2, d, F, 8)):
        most = min(most, 4 * chunk * d // (M * N)) if name != "gu" else 1
        n, rows, _ = ask([("ranges", BF16, nt, M, N, K, max(most, 1))])[0]
        n = n if name != "gu" else 1
        if rows or M <= 32:
            out[name] = ("rows" if rows else "skinny", n, N, K)
        else:
            s = ask([(kind(name == "gu"), BF16, nt, M, N, K, n)])[0][0]
            out[name] = (TILES[s], n, N, K)
    return out


def test_ragged_tile_prompts_reach_every_tile_and_epilogue(ask):
    """What test_ragged_tiles_match_oracle says of its configurations: every tile with
    stored, residual, SwiGLU and K-range results, at a row remainder and a column remainder
    (a SwiGLU product has whole 128-column tiles always)."""
    seen = set()
    for name, sizes in TILE_ROWS.items():
        for M in sizes:
            for p, (tile, n, N, K) in prompt_products(ask, TILE_CFGS[name], M).items():
                if tile not in TILES:
                    continue
                bm, bn = map(int, tile.split("x"))
                what = "ranges" if n > 1 else {"qkv": "store", "gu": "swiglu"}.get(p, "resid")
                if M % bm and (N % bn or (what == "swiglu" and bn == 128)):
                    seen.add((what, tile))
    assert seen == {(w, t) for w in ("store", "resid", "swiglu", "ranges") for t in TILES}


def test_odd_depths_reach_the_other_kernels(ask):
    """K of 64 mod 128: k_gemm_skinny up to 32 rows, tiles from 33."""
    for name in ("odd", "step"):
        for M, want in ((1, "skinny"), (32, "skinny"), (33, "64x128"), (129, "64x128")):
            got = prompt_products(ask, CFGS[name], M)
            assert {v[0] for v in got.values()} == {want}, (name, M, got)
            assert all(v[3] // v[1] % 128 == 64 for v in got.values())
