"""Channel slab and row tiles per workgroup of the step kernels (host arithmetic, compiled on its own: no GPU)."""
import os
import subprocess

import pytest

from util import TWO_LAUNCHES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "step_tiling.h"
// m ntile B kt2 parts elem cus, widest slab, narrow slab -> chunks tiles, the best of 16..6 at the widest slab and its fill
// with an argument: rt kt2 N B cus -> whether the smoothing full step takes rt row tiles; with two: B N D kt2 parts cus ->
// whether the full step takes tiles of 16 rows; with three: B N D k f32 smoothing / tensor added cus -> 10 x the row tiles of the
// general full step in parts + whether the general cached step runs in parts; with four: B N D k f32 states cus -> the latter; with five:
// rows l tiles most cus -> rows of a slice of the Gram matrices; with six: ntile B kt D cus -> whether a projection is large; with
// seven: B N D k f32 split cus -> row tiles of the projection of a full step that takes two launches, or 0; with eight: B N D states cus -> whether a
// cached step that adds a tensor takes slabs of 12 chunks; with nine: B N D k cus -> whether one of two states does not share its coefficients;
// with ten: B N D kt2 f32 split states cus, the widest slab and whether a tensor is added -> the narrow slab, and chunks and tiles of what is launched
int main(int argc, char**) {
  if (argc > 10) {
    long long B;
    int N, D, kt2, f32, split, states, cus, chunks, adds;
    while (std::scanf("%lld %d %d %d %d %d %d %d %d %d", &B, &N, &D, &kt2, &f32, &split, &states, &cus, &chunks, &adds) == 10) {
      const int m = D / 128, narrow = svdc::narrow_slab(m, chunks, kt2, f32, states > 1);
      const svdc::CachedTiling t = svdc::cached_tiling({m, (N + 15) / 16, B, kt2, split ? 2 : 1, f32 ? 4 : 2, cus}, chunks, narrow, adds ? svdc::kAddingOneRound : 0.7);
      std::printf("%d %d %d 0\n", narrow, t.chunks, t.tiles);
    }
    return 0;
  }
  if (argc > 9) {
    long long B;
    int N, D, k, cus;
    while (std::scanf("%lld %d %d %d %d", &B, &N, &D, &k, &cus) == 5) std::printf("%d\n", (int)svdc::two_states_stay_unshared((N + 15) / 16, B, D, k, cus));
    return 0;
  }
  if (argc > 8) {
    long long B;
    int N, D, states, cus;
    while (std::scanf("%lld %d %d %d %d", &B, &N, &D, &states, &cus) == 5)
      std::printf("%d\n", (int)svdc::adding_takes_wide_slabs({D / 128, (N + 15) / 16, B, 1, 2, 2, cus}, states));
    return 0;
  }
  if (argc > 7) {
    long long B;
    int N, D, k, f32, split, cus;
    while (std::scanf("%lld %d %d %d %d %d %d", &B, &N, &D, &k, &f32, &split, &cus) == 7)
      std::printf("%d\n", svdc::full_step_projection_rows(N, B, D, k, f32, split, cus));
    return 0;
  }
  if (argc > 6) {
    long long B;
    int ntile, kt, D, cus;
    while (std::scanf("%d %lld %d %d %d", &ntile, &B, &kt, &D, &cus) == 5) std::printf("%d\n", (int)svdc::projection_is_large(ntile, B, kt, D, cus));
    return 0;
  }
  if (argc > 5) {
    int rows, l, cus;
    long long tiles, most;
    while (std::scanf("%d %d %lld %lld %d", &rows, &l, &tiles, &most, &cus) == 5)
      std::printf("%d\n", svdc::gram_slice_rows(rows, l, tiles, most, cus));
    return 0;
  }
  if (argc > 4) {
    int N, D, k, f32, states, cus;
    long long B;
    while (std::scanf("%lld %d %d %d %d %d %d", &B, &N, &D, &k, &f32, &states, &cus) == 7)
      std::printf("%d\n", (int)(svdc::cached_step_may_take_parts(D, k, f32, states, false) &&
                                svdc::cached_step_takes_parts(N, B, D, k, f32, states, cus)));
    return 0;
  }
  if (argc > 3) {
    int N, D, k, f32, extra, cus;
    long long B;
    while (std::scanf("%lld %d %d %d %d %d %d", &B, &N, &D, &k, &f32, &extra, &cus) == 7)
      std::printf("%d\n", (svdc::full_step_may_take_parts(D, k, f32, extra) ? 10 * svdc::full_step_parts_rows(N, B, D, k, f32, extra, cus) : 0) +
                               (svdc::cached_step_may_take_parts(D, k, f32, 1, extra) && svdc::cached_step_takes_parts(N, B, D, k, f32, 1, cus)));
    return 0;
  }
  if (argc > 2) {
    long long B, N, D, kt2, parts, cus;
    while (std::scanf("%lld %lld %lld %lld %lld %lld", &B, &N, &D, &kt2, &parts, &cus) == 6)
      std::printf("%d\n", (int)svdc::full_step_takes_single_tiles((N + 15) / 16 * B, B * D * 32 * kt2 * 2 * parts, (int)cus));
    return 0;
  }
  if (argc > 1) {
    int rt, kt2, N, cus;
    long long B;
    while (std::scanf("%d %d %d %lld %d", &rt, &kt2, &N, &B, &cus) == 5)
      std::printf("%d\n", (int)svdc::smoothing_takes_full_tiles(rt, kt2, N, B, cus));
    return 0;
  }
  svdc::CachedCall c;
  long long B;
  int chunks, narrow;
  while (std::scanf("%d %d %lld %d %d %d %d %d %d", &c.m, &c.ntile, &B, &c.kt2, &c.parts, &c.elem, &c.cus, &chunks, &narrow) == 9) {
    c.B = B;
    const svdc::CachedTiling t = svdc::cached_tiling(c, chunks, narrow);
    int best = 16;
    for (int n = 15; n >= 6; --n)
      if (c.fill({chunks, n}) > c.fill({chunks, best}) + 1e-9) best = n;
    std::printf("%d %d %d %.9f\n", t.chunks, t.tiles, best, c.fill({chunks, best}));
  }
}
"""


@pytest.fixture(scope="module")
def tiling(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiling")
    src, exe = str(d / "tiling.cpp"), str(d / "tiling")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2601_07396_amd", "csrc"), "-o", exe,
                    src], check=True)

    def run(calls, rule=()):
        text = "\n".join(" ".join(str(int(x)) for x in c) for c in calls)
        out = subprocess.run([exe, *rule], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout
        if len(rule) in (5, 7):
            return [int(line) for line in out.split()]
        if len(rule) == 3:
            return [(int(line) // 10, bool(int(line) % 10)) for line in out.split()]
        if rule and len(rule) != 10:
            return [bool(int(line)) for line in out.split()]
        return [(int(a), int(b), int(c), float(d)) for a, b, c, d in (line.split() for line in out.splitlines())]
    return run


def _narrow(m, chunks):
    return 0 if chunks <= 3 else (3 if m % 3 == 0 else (2 if m % 2 == 0 else 0))


def _calls():
    for m in (2, 4, 8, 9, 12, 15, 16, 20, 24, 32, 40):
        for chunks in (1, 2, 3, 4, 6, 8, 9, 12):
            if m % chunks:
                continue
            for B in (1, 2, 4, 19, 28, 57, 300):
                for ntile in (1, 2, 5, 13, 42, 63, 125, 288, 423, 1152, 7441):
                    for kt2, parts, elem in ((1, 2, 2), (2, 1, 2), (4, 2, 2), (4, 2, 4)):
                        for cus in (32, 256):
                            yield m, ntile, B, kt2, parts, elem, cus, chunks, _narrow(m, chunks)


def test_a_call_that_fills_the_machine_reuses_its_basis(tiling):
    """Every workgroup loads the basis operands of its slab once and uses them for each of its row tiles.  Fewer than six
    tiles are for calls that leave the machine unfilled otherwise, whatever the width of the slab; in a call that fills it
    they trade basis traffic for a rounder grid."""
    calls = list(_calls())
    filled = 0
    for call, (chunks, tiles, tiles6, fill6) in zip(calls, tiling(calls)):
        assert call[0] % chunks == 0 and 1 <= tiles <= 16, call
        if fill6 >= 0.7:
            filled += 1
            assert (chunks, tiles) == (call[7], tiles6), call
        elif tiles < 6:
            assert chunks <= 3 and tiles <= call[1], call
    assert filled > 1000


@pytest.mark.parametrize("m,ntile,B,kt2,parts,elem,chunks,tiles", [
    (24, 7442, 2, 2, 2, 2, 3, 13), (24, 125, 24, 2, 2, 2, 3, 16), (24, 125, 24, 4, 2, 2, 1, 7), (9, 288, 57, 4, 2, 2, 3, 9),
    (2, 7442, 2, 1, 2, 2, 2, 15), (15, 97, 28, 4, 2, 4, 1, 7)])
def test_large_calls_with_slabs_of_at_most_three_chunks(tiling, m, ntile, B, kt2, parts, elem, chunks, tiles):
    """Several-state forecasts and cached steps for which three chunks or fewer are the widest slab: 2 x 119056 and 24 x 2000
    rows of 3072 channels at rank 64 and 128, 57 x 4608 x 1152, 2 x 119056 x 256, 28 x 1548 x 1920 in float32."""
    assert tiling([(m, ntile, B, kt2, parts, elem, 256, chunks, 0)])[0][:2] == (chunks, tiles)


def test_small_calls(tiling):
    """A single block of 4608 x 3072 takes narrow slabs; blocks of a few rows at rank 128, whose basis operands outweigh their
    features, stay on the widest one."""
    assert tiling([(24, 288, 1, 1, 2, 2, 256, 12, 3)])[0][0] == 3
    assert tiling([(24, 288, 1, 2, 2, 2, 256, 8, 3)])[0][0] == 3
    assert tiling([(16, 9, 43, 4, 2, 2, 256, 4, 2)])[0][0] == 4
    chunks, tiles = tiling([(15, 8, 19, 4, 2, 2, 256, 3, 0)])[0][:2]
    assert chunks == 3 and 5 * 19 * -(-8 // tiles) <= 256     # 19 blocks of 128 x 1920: one round, not three with one tile each


def test_smoothing_full_step_takes_the_taller_tile_where_it_saves_time(tiling):
    """Measured (us with the taller tile, with one less).  64 rows: 1 x 96983 x 512 rank 8 single operands 69.8 / 66.0,
    1 x 52658 x 256 rank 48 35.0 / 33.5, 19 x 17388 x 512 rank 8 233.8 / 225.7; 28 x 1024 x 1152 rank 32 57.7 / 60.7.
    32 rows at rank 128: 19 x 352 x 1024 33.8 / 38.8, 19 x 751 x 1024 36.6 / 47.5."""
    calls = [(4, 1, 96983, 1), (4, 2, 52658, 1), (4, 1, 17388, 19), (4, 1, 1024, 28), (2, 4, 352, 19), (2, 4, 751, 19)]
    assert tiling([c + (256,) for c in calls], rule=["smoothing"]) == [False, False, False, True, True, True]


def test_small_full_steps_take_single_tiles_while_l2_holds_the_basis(tiling):
    """Measured (us with 16-row tiles, with tiles one step below the full height): 4 x 700 x 3072 rank 32 17 / 23, 28 x 128 x 1152
    rank 32 single operands 8.7 / 11.0, 57 x 32 x 3072 rank 32 20.2 / 22.9; 28 x 125 x 1152 rank 64 22.3 / 18.2, 26 x 128 x 1920
    rank 64 33.2 / 23.4, 57 x 48 x 512 rank 64 11.0 / 9.9; 4608 x 3072 rank 32 does not fit one round."""
    calls = [(4, 700, 3072, 1, 2), (28, 128, 1152, 1, 1), (57, 32, 3072, 1, 2),
             (28, 125, 1152, 2, 2), (26, 128, 1920, 2, 2), (57, 48, 512, 2, 2), (1, 4608, 3072, 1, 2)]
    assert tiling([c + (256,) for c in calls], rule=["full", "step"]) == [True, True, True, False, False, False, False]


def test_general_steps_in_parts(tiling):
    """Row tiles of the general full step on the bf16 matrix cores (0: the float32 ones) and whether the cached step runs there:
    the sizes of the GPU tests, measured ones (gain), and the limits of the rank, the channels, the rows and the storage type."""
    want = [((1, 601, 2008, 64, 0, 0), (1, False)), ((1, 8101, 520, 50, 0, 0), (2, False)), ((1, 8701, 520, 50, 0, 0), (3, False)),
            ((1, 8101, 1288, 50, 0, 0), (2, True)), ((1, 8701, 800, 50, 1, 0), (3, False)), ((1, 6001, 1036, 117, 1, 0), (2, True)),
            ((1, 8701, 776, 50, 0, 1), (3, False)), ((1, 4931, 1168, 86, 0, 1), (2, False)), ((1, 3517, 2056, 121, 0, 0), (1, True)),
            ((4, 2173, 1408, 50, 0, 0), (3, True)), ((6, 700, 3304, 33, 0, 0), (2, True)), ((1, 1500, 1304, 100, 0, 0), (1, False)),
            ((17, 230, 616, 24, 0, 0), (0, False)), ((15, 258, 1000, 72, 1, 0), (0, False)), ((3, 4082, 888, 34, 0, 1), (0, False)),
            ((20, 900, 1000, 16, 0, 0), (0, False)), ((57, 3874, 72, 36, 0, 0), (0, False)), ((4, 2173, 1408, 129, 0, 0), (0, False)),
            ((1, 8701, 800, 50, 1, 1), (0, False)), ((1, 10032, 2800, 9, 1, 0), (0, False))]
    assert tiling([c + (256,) for c, _ in want], rule=["general", "steps", "parts"]) == [w for _, w in want]


def test_general_cached_steps_of_several_states_in_parts(tiling):
    """Several states have to promise more; those of float32 rows stay on the float32 instructions."""
    calls = [(1, 3517, 2056, 121, 0, 2), (1, 8101, 1288, 50, 0, 4), (4, 1292, 976, 128, 0, 1), (4, 1292, 976, 128, 0, 2),
             (1, 6001, 1036, 117, 1, 1), (1, 6001, 1036, 117, 1, 2)]
    assert tiling([c + (256,) for c in calls], rule=["cached", "steps", "of", "states"]) == [True, True, True, False, True, False]


def test_slices_of_the_gram_matrices(tiling):
    """Above 64 columns a compute unit holds one workgroup: 3 x 5120 rows take 54 slices (486 workgroups) 25 us and 27 slices (243) 17, 4 x
    14777 rows 24 slices (288) 56 us and 21 (252) 43, 20 x 3000 8 slices 46 and 4 41.  One block takes all that the workspace holds.  Up to 64 three fit."""
    calls = [(5120, 128, 9, 100), (9179, 128, 9, 53), (14777, 128, 12, 24), (3000, 128, 60, 40), (18432, 128, 3, 40), (4608, 64, 57, 40), (33, 70, 3, 16)]
    assert tiling([c + (256,) for c in calls], rule=["slices", "of", "the", "Gram", "matrices"]) == [192, 336, 704, 752, 464, 368, 64]
    many = [(rows, l, tiles, most) for rows in (1, 63, 65, 1000, 18432) for l in (1, 64, 65, 256) for tiles in (1, 10, 300, 70000)
            for most in (1, 16, 400)]
    for (rows, _, _, most), r in zip(many, tiling([c + (256,) for c in many], rule=["slices", "of", "the", "Gram", "matrices"])):
        assert r >= 64 and r % 16 == 0 and -(-rows // r) <= most


def test_wide_projections_that_do_not_stream(tiling):
    """Measured (us of the plain product, kernel that shares Q and streamed): 4 x 14777 x 1024 width 128 28 / 43, 34 x 1264 x 512 17 / 26; whole fits: 15 x 3837 x
    768 width 72 767 / 818, 4 x 15877 x 4096 1918 / 2049; 2 x 17284 x 2560 width 100 1164 / 1107, 44 x 1417 x 1920 width 80 1714 / 1662 (528 workgroups).
    Width 64 streams up to 16 tiles per unit."""
    calls = [((924, 4, 8, 1024), True), ((79, 34, 8, 512), True), ((240, 15, 8, 768), True), ((993, 4, 8, 4096), True), ((1081, 2, 8, 2560), False),
             ((89, 44, 8, 1920), False), ((182, 20, 4, 2560), False), ((288, 57, 4, 3072), True), ((30, 57, 8, 1024), False), ((2047, 1, 8, 1024), False),
             ((2048, 1, 8, 1024), True), ((3071, 1, 8, 1152), False), ((3072, 1, 8, 1152), True), ((4095, 1, 4, 512), False), ((4096, 1, 1, 512), True)]
    assert tiling([c + (256,) for c, _ in calls], rule=["which", "projections", "of", "a", "fit", "stream"]) == [w for _, w in calls]


def test_full_steps_in_two_launches(tiling):
    """The calls of the GPU test of the two launches take them, at every height of the projection's tiles, and so do 18432 x 3072 float32 at rank 128 (235 us in one
    launch, 190 in two) and 57 x 4608 x 3072 bf16 (2117 / 1645); not at rank 64 (1174 / 1223) and 32 (871 / 1020), nor in single operands at rank 64."""
    rule = ["which", "full", "steps", "take", "two", "launches", "instead"]
    calls = [(B, N, D, k, dtype == "f32", not fast, 256) for dtype, B, N, D, k, fast, _, _ in TWO_LAUNCHES]
    assert tiling(calls, rule=rule) == [c[7] for c in TWO_LAUNCHES] and {c[7] for c in TWO_LAUNCHES} == {1, 2, 3, 4, 5, 6}
    calls = [(1, 18432, 3072, 128, 1, 1), (57, 4608, 3072, 128, 0, 1), (57, 4608, 3072, 64, 0, 1), (57, 4608, 3072, 32, 0, 1), (2, 119056, 3072, 64, 0, 0),
             (1, 300, 256, 128, 1, 1), (4, 2048, 4096, 32, 1, 1)]
    assert [r > 0 for r in tiling([c + (256,) for c in calls], rule=rule)] == [True, True, False, False, False, False, False]


@pytest.mark.parametrize("ntile,B,rows", [(1, 1, 1), (256, 1, 1), (257, 1, 2), (288, 1, 2), (1000, 1, 4), (1152, 1, 5), (288, 20, 6), (288, 4, 5)])
def test_heights_of_the_streamed_projection(tiling, ntile, B, rows):
    """Rounds x (rows + 1.25) is least: 1152 tiles are 231 workgroups of 5 (one round); of 6 192, of 4 288, two rounds."""
    assert tiling([(B, 16 * ntile, 4096, 128, 1, 1, 256)], rule=["which", "full", "steps", "take", "two", "launches", "instead"]) == [rows]


def test_cached_steps_that_add_a_tensor_in_wide_slabs(tiling):
    """Measured (us with slabs of 12 chunks, with 6 shared): 57 x 4608 x 3072 rank 32 two states 945 / 969, 19 x 4608 x 3072 327 / 323,
    6 x 4608 x 3072 108 / 104, four states in 3 rounds of the narrower slabs 4 x 6865 x 3072 1 / 1.11 of its time.  Not for widths that 12 chunks do not divide."""
    calls = [((57, 4608, 3072, 2), True), ((57, 4608, 3072, 4), True), ((19, 4608, 3072, 2), False), ((6, 4608, 3072, 2), False),
             ((4, 6865, 3072, 4), True), ((4, 6865, 3072, 2), False), ((1, 85001, 3072, 2), True), ((8, 5206, 1536, 3), True), ((1, 300, 3072, 4), False), ((57, 4608, 2048, 2), False), ((57, 4608, 5120, 4), False)]
    rule = ["which", "cached", "steps", "that", "add", "take", "wide", "slabs"]
    assert tiling([c + (256,) for c, _ in calls], rule=rule) == [w for _, w in calls]


def test_cached_steps_of_two_states_that_do_not_share(tiling):
    """Measured (us unshared, shared): 4 x 12079 x 4096 rank 8 165 / 176, 6 x 21312 x 2048 rank 16 217 / 230, 41 x 4525 x 1024 rank 8 172 / 181; with a rank above 16,
    other widths and shorter calls the shared ones are faster."""
    calls = [((4, 12079, 4096, 8), True), ((6, 21312, 2048, 16), True), ((41, 4525, 1024, 8), True), ((1, 308001, 512, 4), True), ((6, 21312, 2048, 20), False),
             ((57, 4608, 3072, 8), False), ((57, 4608, 1152, 8), False), ((4, 6000, 4096, 8), False)]
    rule = ["which", "cached", "steps", "of", "two", "states", "do", "not", "share"]
    assert tiling([c + (256,) for c, _ in calls], rule=rule) == [w for _, w in calls]


@pytest.mark.parametrize("B,N,D,kt2,f32,split,states,widest,want", [
    (1, 439, 1152, 4, 1, 1, 1, 3, (1, 1)), (1, 18432, 1152, 4, 1, 1, 1, 3, (1, 3)),       # rank 128, 9 chunks: one chunk in a short call, 3 in a long one
    (1, 273, 1152, 2, 1, 1, 2, 3, (1, 1)), (1, 304, 256, 2, 1, 1, 2, 2, (1, 1)), (2, 404, 512, 4, 1, 1, 2, 2, (1, 1)), (1, 336, 512, 2, 1, 1, 2, 4, (1, 1)),
    (1, 18432, 3072, 2, 1, 1, 2, 3, (1, 3)), (28, 1548, 1920, 4, 1, 1, 1, 3, (1, 3)), (1, 273, 1152, 2, 1, 1, 1, 3, (0, 3)),
    (24, 2000, 3072, 2, 0, 1, 2, 4, (3, 4)), (2, 119056, 3072, 4, 0, 1, 2, 2, (0, 2)), (1, 4608, 3072, 1, 0, 1, 1, 12, (3, 3)), (1, 4608, 2048, 1, 0, 1, 1, 8, (2, 2))])
def test_slabs_of_the_cached_step(tiling, B, N, D, kt2, f32, split, states, widest, want):
    """With the widest slab that the launcher starts from: the narrower one that it may take, and the one that it takes.  One chunk in the place of 3 or 2
    where float32 rows have several states (us: 1 x 273 x 1152 rank 48 5.1 -> 3.7, 2 x 404 x 512 rank 124 4.6 -> 4.0)."""
    rule = ["which", "slabs", "does", "the", "cached", "step", "take", "in", "the", "end"]
    assert tiling([(B, N, D, kt2, f32, split, states, 256, widest, 0)], rule=rule)[0][:2] == want


@pytest.mark.parametrize("B,N,D,widest,plain,adding", [(12, 749, 1536, 6, 6, 3), (8, 534, 2048, 4, 4, 2), (1, 4368, 3072, 6, 6, 3), (6, 4608, 3072, 6, 6, 6), (1, 5400, 3072, 6, 6, 6)])
def test_cached_steps_that_add_a_tensor_fill_one_round(tiling, B, N, D, widest, plain, adding):
    """Two workgroups of these steps fit on a compute unit: a grid of at most one per unit that fills less than 0.9 of that gives way to narrower slabs.  Measured (us with the
    slab that others keep, with the narrower one): 12 x 749 x 1536 four states 25.6 / 23.3, 8 x 534 x 2048 two states 16.5 / 15.2, 1 x 4368 x 3072 24.5 / 21.1."""
    rule = ["which", "slabs", "does", "the", "cached", "step", "take", "in", "the", "end"]
    got = tiling([(B, N, D, 1, 0, 1, 2, 256, widest, adds) for adds in (0, 1)], rule=rule)
    assert [g[1] for g in got] == [plain, adding]


def test_full_steps_of_more_rows_than_a_grid_has_workgroups_stay_one_launch(tiling):
    """The single launch refuses those before anything runs; the projection of two launches has no such check of its own."""
    rule = ["which", "full", "steps", "take", "two", "launches", "instead"]
    calls = [(170, 2 ** 30 - 1, 1536, 128, 0, 1, 256), (3, 2 ** 30 - 1, 5120, 8, 1, 1, 256), (60, 119056, 3072, 128, 0, 1, 256)]
    assert [r > 0 for r in tiling(calls, rule=rule)] == [False, False, True]
