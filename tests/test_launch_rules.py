"""Host-side rules behind the launches, compiled from their headers with the host compiler (no GPU)."""
import ctypes
import glob
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_05346_amd", "csrc")


def _compile(tmp_path_factory, name, source):
    d = tmp_path_factory.mktemp(name)
    src, lib = d / f"{name}.cpp", d / f"lib{name}.so"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)],
                   check=True)
    return ctypes.CDLL(str(lib))


@pytest.fixture(scope="module")
def lam(tmp_path_factory):
    L = _compile(tmp_path_factory, "lam", """
#include "lam_layout.h"
extern "C" void offsets(int64_t c, int64_t ldl, int64_t sbi, int64_t* o) {
  const thanos::LamLayout l = thanos::lam_layout(c, ldl, sbi);
  o[0] = l.lam, o[1] = l.z, o[2] = l.wk;
}
extern "C" int64_t buffer(int64_t c, int64_t B) { return thanos::lam_buffer_floats(c, B); }
extern "C" int64_t super() { return thanos::kSuper; }
""")
    L.offsets.argtypes = [ctypes.c_int64] * 3 + [ctypes.POINTER(ctypes.c_int64)]
    L.buffer.argtypes = [ctypes.c_int64] * 2
    L.buffer.restype = L.super.restype = ctypes.c_int64
    return L


@pytest.mark.parametrize("c,B", [(2560, 256), (2603, 132), (16640, 512), (1 << 24, 512)])
def test_multipliers_and_complement_operands_are_disjoint(lam, c, B):
    """Unstructured sweep (a super-block is one block): the multipliers of a block of either parity
    and the operands Z and WK of the complement products share no memory and lie in the buffer."""
    for blk in range(4):
        o = (ctypes.c_int64 * 3)()
        lam.offsets(c, B, blk, o)
        starts = sorted(o)
        assert starts[0] >= 0
        assert all(b - a >= c * B for a, b in zip(starts, starts[1:])), (blk, list(o))
        assert starts[-1] + c * B <= lam.buffer(c, B)


def test_multipliers_of_consecutive_super_blocks_are_disjoint(lam):
    c, B = 4097, 128
    ldl = B * lam.super()
    o = [(ctypes.c_int64 * 3)() for _ in range(2)]
    for sbi in range(2):
        lam.offsets(c, ldl, sbi, o[sbi])
    assert abs(o[0][0] - o[1][0]) >= c * ldl
    assert max(o[0][0], o[1][0]) + c * ldl <= lam.buffer(c, B)


# --------------------------------------------------------------------------- LDS limits
def test_a_kernels_lds_limit_is_one_constant():
    """The limit of a kernel is state of the process: two calls that set it to different values can come
    between each other's setting and launch.  So it is a constant, or a value that goes with the
    kernel (chosen in one statement with it, or computed from its template arguments)."""
    found = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        text = open(path).read()
        for m in re.finditer(r"hipFuncSetAttribute\(reinterpret_cast<const void\*>\((.*?)\),\s*"
                             r"hipFuncAttributeMaxDynamicSharedMemorySize,\s*\(int\)(\w+)", text):
            kernel, value = m.groups()
            found += 1
            if value != "smem":
                assert re.match(r"k[A-Z]|tl_big_smem_bytes", value), (path, kernel, value)
            elif kernel == "kern":
                before = text[:m.start()]
                choices = re.findall(r"kern = .*? : .*?, smem = ([\w<>:]+)[;,]", before[before.rindex("void (*kern)"):])
                assert choices and all(re.match(r"k[A-Z]\w*(<|$)|DmaCfg<", c) for c in choices), (path, choices)
            else:  # k_solve_mfma<.., WPB, NTR>
                last = re.findall(r"smem = (.*?);", text[:m.start()])[-1]
                assert re.fullmatch(r"\w+ \* sizeof\(SolveMfmaSmem<\d>\)", last), (path, last)
    assert found >= 10


# --------------------------------------------------------------------------- 16-bit Hessian accumulation
class Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("tile", "nt", "ntiles", "nkt", "nsplit", "spread")] + [
        ("grid", ctypes.c_uint)]


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    L = _compile(tmp_path_factory, "plan", """
#include "syrk_plan.h"
extern "C" void plan(int64_t b, int64_t n_tok, int aligned, thanos::SyrkPlan* p) {
  *p = thanos::syrk_plan(b, n_tok, aligned != 0);
}
extern "C" int aligned(uintptr_t X, int64_t ldx, int64_t b) { return thanos::syrk_rows_aligned(X, ldx, b); }
extern "C" int64_t launch_tokens(int64_t b, int64_t n_tok) { return thanos::syrk_launch_tokens(b, n_tok); }
extern "C" int64_t round_parts(int64_t b, int64_t n_tok) { return thanos::round_parts(b, n_tok); }
""")
    L.plan.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.POINTER(Plan)]
    L.round_parts.argtypes = [ctypes.c_int64, ctypes.c_int64]
    L.round_parts.restype = ctypes.c_int64
    L.launch_tokens.argtypes = [ctypes.c_int64, ctypes.c_int64]
    L.launch_tokens.restype = ctypes.c_int64
    L.aligned.argtypes = [ctypes.c_size_t, ctypes.c_int64, ctypes.c_int64]

    def call(b, n_tok, aligned):
        p = Plan()
        L.plan(b, n_tok, int(aligned), ctypes.byref(p))
        return p
    call.round_parts, call.aligned, call.launch_tokens = L.round_parts, L.aligned, L.launch_tokens
    return call


CHANNELS = [8, 64, 237, 256, 512, 700, 768, 1024, 1365, 2048, 2816, 2817, 3001, 4096, 5121, 8191, 11008, 28672]
TOKENS = [1, 31, 512, 2048, 5065, 16384, 65536, 262144]


@pytest.mark.parametrize("aligned", [False, True])
def test_every_part_of_every_tile_has_one_workgroup(plan, aligned):
    """The dealing of item_of (syrk.hip): each (tile, part) exactly once."""
    for b in CHANNELS:
        for T in TOKENS:
            p = plan(b, T, aligned)
            assert p.nt == -(-b // p.tile) and p.ntiles == p.nt * (p.nt + 1) // 2
            seen = set()
            for wg in range(p.grid):
                xcd, local = wg & 7, wg >> 3
                if p.spread:
                    r = xcd * (p.grid >> 3) + local
                    part, tile, cnt = r // p.ntiles, r % p.ntiles, 1
                else:
                    cnt = p.ntiles // 8 + (1 if xcd < p.ntiles % 8 else 0)
                    part = local // max(cnt, 1)
                    tile = xcd * (p.ntiles // 8) + min(xcd, p.ntiles % 8) + local - part * cnt
                if cnt > 0 and part < p.nsplit:
                    assert (tile, part) not in seen and 0 <= tile < p.ntiles
                    seen.add((tile, part))
            assert len(seen) == p.ntiles * p.nsplit, (b, T)


def test_row_offsets_of_the_loads_to_lds_fit_32_bits(plan):
    """A wavefront reaches eight rows (two per load) from one descriptor: 7 ldx + b two-byte elements."""
    assert plan.aligned(4096, 4104, 4096) and not plan.aligned(4098, 4104, 4096)
    assert not plan.aligned(4096, 4097, 4096) and not plan.aligned(4096, 4104, 4095)
    for ldx in (1 << 20, (1 << 28) - 8, 1 << 28, 306783376, 1 << 29, 1 << 33):
        if plan.aligned(4096, ldx, 4096):
            assert 2 * (7 * ldx + 4096) < 1 << 32, ldx
    assert plan.aligned(4096, (1 << 28) - 8, 4096)


def test_rows_of_any_alignment_are_summed_up_in_one_part(plan):
    for b in CHANNELS:
        for T in TOKENS:
            assert plan(b, T, False).nsplit == 1


def test_sums_over_rows_of_any_alignment_are_short(plan):
    """At most 4096 tokens in any one sum (8192 in a 256-wide tile), in launches that cover the call."""
    for b in CHANNELS:
        for T in TOKENS + [8193, 32769, 65537]:
            n = plan.launch_tokens(b, T)
            assert 0 < n and n % 128 == 0
            p = plan(b, min(n, T), False)
            sums = {32: 16, 64: 8, 128: 2, 256: 1}[p.tile]
            assert n <= 8192 if p.tile == 256 else n <= 4096 * sums, (b, T)


def test_old_values_are_read_from_inside_h(tmp_path_factory, plan):
    """What the accumulation reads of H around each 32 x 32 part of a tile ends with H, whatever the size leaves of
    the last tile, and holds all that the part adds to."""
    L = _compile(tmp_path_factory, "window", """
#include "syrk_plan.h"
// parts of the tiles of one row of tiles; 0, or 1 + the first part that reads outside of H or lacks a value
extern "C" int64_t check(int64_t b, int64_t tile, int64_t ti) {
  int64_t n = 0;
  for (int64_t tj = 0; tj <= ti; tj += tj + 2 < ti ? ti - 1 - tj : 1)  // the first, the last two
    for (int64_t i0 = ti * tile; i0 < (ti + 1) * tile; i0 += 32)
      for (int64_t j0 = tj * tile; j0 < (tj + 1) * tile; j0 += 32) {
        ++n;
        const thanos::HWindow w = thanos::h_window(b, i0, j0);
        if (w.first < 0 || 4 * (__int128)w.first + w.bytes > 4 * (__int128)b * b) return n;
        for (int64_t i = i0; i < i0 + 32 && i < b; ++i) {
          const int64_t j = i < j0 + 31 ? i : j0 + 31;  // the last value of the row that is added to
          if (j >= j0 && (w.first != i0 * b + j0 || 4 * ((i - i0) * b + j - j0) + 4 > w.bytes)) return n;
        }
      }
  return 0;
}
""")
    L.check.argtypes = [ctypes.c_int64] * 3
    L.check.restype = ctypes.c_int64
    sizes = list(range(1409, 1409 + 768)) + [4001, 5121, 8193, 11008, 28672, 28673, 65505, 65535]
    for b in sizes:
        for tile in (128, 192, 256):
            nt = -(-b // tile)
            for ti in (0, nt // 2, nt - 1):
                assert L.check(b, tile, ti) == 0, (b, tile, ti)


def test_few_channels_take_narrow_tiles(plan):
    """The 32- and 64-wide tiles are for calls whose tiles run all at once, in one part."""
    for b in CHANNELS + [704, 705, 1408, 1409]:
        for T in TOKENS:
            for aligned in (False, True):
                p = plan(b, T, aligned)
                if p.tile < 128:
                    assert p.ntiles <= 256 and p.nsplit == 1 and p.spread
                    assert p.nkt * (32768 // p.tile) >= T
                else:
                    assert b > 1408 or (aligned and T > 4064), (b, T)


def test_aligned_rows_are_cut_into_parts_for_whole_rounds_only(plan):
    """Up to 4064 tokens: one part.  More: no more parts than fill rounds of 256-wide tiles, and
    sums no longer than theirs (two groups of wavefronts halve a part of the narrower tiles)."""
    for b in CHANNELS:
        assert all(plan(b, T, True).nsplit == 1 for T in TOKENS + [4064] if T <= 4064)
        for T in TOKENS:
            p = plan(b, T, True)
            assert p.nsplit <= plan.round_parts(b, T), (b, T)
            assert p.nsplit * (1 if p.tile == 256 else 2) >= plan.round_parts(b, T), (b, T)


def test_shapes_of_the_gpu_tests_reach_every_tile_width(plan):
    from tests.test_gpu_hessian import WIDTHS
    for b, T, width in WIDTHS:
        assert plan(b, T, b % 8 == 0).tile == width, (b, T)


def test_row_scales_lie_behind_the_complement_operands(tmp_path_factory):
    """Unstructured: one block per super-block; the scales of the rows share nothing with the two slices of
    multipliers or with the operands of the complement products, and fit the buffer."""
    L = _compile(tmp_path_factory, "rsc", """
#include "lam_layout.h"
extern "C" int ok(int64_t c, int64_t B) {
  for (int64_t sbi = 0; sbi < 3; ++sbi) {
    const thanos::LamLayout l = thanos::lam_layout(c, B, sbi);
    const int64_t n = c * B;
    if (l.rsc < l.lam + n || l.rsc < l.z + n || l.rsc < l.wk + n) return 0;
    if (l.rsc + c > thanos::lam_buffer_floats(c, B)) return 0;
  }
  return 1;
}
""")
    L.ok.argtypes = [ctypes.c_int64] * 2
    for c, B in ((1, 1), (7, 3), (2560, 256), (8192, 512), (1 << 24, 1)):
        assert L.ok(c, B) == 1


def test_split_scales(tmp_path_factory):
    """Scales of the two-way split: powers of two with finite inverses for every bound; bounded values
    times their scale stay below 2^15, columns below 1."""
    L = _compile(tmp_path_factory, "scales", """
#include <cstdint>
#define __host__
#define __device__
#include "split_scale.h"
extern "C" float h2(float x) { return thanos::h2_scale(x); }
extern "C" float col(float x) { return thanos::col_scale(x); }
""")
    for f in (L.h2, L.col):
        f.argtypes, f.restype = [ctypes.c_float], ctypes.c_float
    import math
    for e in range(-149, 128):
        for x in (math.ldexp(1.0, e), math.ldexp(1.9999, e)):
            h, c = L.h2(x), L.col(x)
            assert math.frexp(h)[0] == math.frexp(c)[0] == 0.5
            assert -126 <= math.frexp(h)[1] - 1 <= 126 and -100 <= math.frexp(c)[1] - 1 <= 100
            if -112 <= e <= 127:
                assert 2.0 ** 14 <= x * h <= 2.0 ** 15
            if -100 <= e <= 98:
                assert 0.5 <= x * c < 1.0
    assert L.h2(0.0) == 2.0 ** 126 and L.col(0.0) == 1.0


@pytest.mark.parametrize("rows,b,need,lanes", [
    ([768] * 3, 768, 12 << 20, 3), ([17, 400], 512, 4 << 20, 2), ([2000, 1900], 512, 20 << 20, 1),
    ([64] * 60, 8192, 270 << 20, 4),       # many experts: four workspaces, not sixty
    ([128] * 30, 8192, 275 << 20, 4), ([500] * 4, 5120, 300 << 20, 2), ([768] * 3, 768, 80 << 20, 1),
    ([64] * 3, 8200, 270 << 20, 1), ([64], 512, 1 << 20, 1),
    ([256] * 3, 255, 1 << 20, 1), ([256] * 3, 256, 1 << 20, 3)])  # one block and a little, two blocks
def test_layer_sets_run_few_sweeps_at_once(rows, b, need, lanes):
    """Streams and workspaces of a layer set are bounded whatever the number of matrices: at most four, the
    further ones in no more memory than the factorisation had, and 64 MiB."""
    from paper_2504_05346_amd.layer_set import _lanes
    freed = 3 * 4 * b * b
    got = _lanes(rows, b, 128, need, freed, 256)
    assert got == lanes
    assert (got - 1) * need <= freed + (64 << 20)


def test_selections_side_by_side_are_as_small_as_one(tmp_path_factory):
    """Sweeps that run at the same time: the workgroups of their selections, which wait for each other, are
    together no more than those of the largest of them, so that two sets at once are no closer to the number of
    compute units than two sweeps; a single workgroup waits for nobody.  One call alone: a workgroup per 16
    rows, at most one per unit."""
    from paper_2504_05346_amd.layer_set import _lanes
    L = _compile(tmp_path_factory, "select", """
#include "select_plan.h"
extern "C" int wgs(int64_t c, int units, int sharers) { return thanos::select_workgroups(c, units, sharers); }
""")
    L.wgs.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    for c in (1, 16, 17, 768, 3840, 4096, 28672, 1 << 24):
        for units in (32, 256, 304):
            assert L.wgs(c, units, 1) == min(-(-c // 16), units, 256)
    for rows in ([768] * 3, [17, 400], [1280] * 3, [64] * 60, [3000, 100, 200], [16, 32, 48, 8], [1920, 1920]):
        lanes = _lanes(rows, 512, 128, 1 << 20, 1 << 30, 256)
        assert lanes == min(4, len(rows))
        at_once = sorted((L.wgs(c, 256, lanes) for c in rows), reverse=True)[:lanes]
        assert sum(n for n in at_once if n > 1) <= max(L.wgs(c, 256, 1) for c in rows)


# --------------------------------------------------------------------------- factorisation
@pytest.fixture(scope="module")
def order(tmp_path_factory):
    L = _compile(tmp_path_factory, "factor_plan", """
#include "factor_plan.h"
extern "C" int first_step(int nb) { return thanos::factor_first_step(nb); }
extern "C" int rests(int nb) { return thanos::factor_rests(nb); }
extern "C" int tri_batches(int nb) { return thanos::factor_tri_batches(nb); }
""")
    return L


def test_steps_follow_whole_outer_blocks(order):
    """Up to 32 block columns are left with one launch per step from the first one on; of more, two-level updates come
    first, in outer blocks of four, and both block columns behind the last of these and rows for its rest are there."""
    for nb in range(1, 513):
        first = order.first_step(nb)
        if nb <= 32:
            assert first == 0
        else:
            assert first > 0 and first % 4 == 0 and 21 <= nb - first <= 24, nb


def test_factorisation_borrows_the_helpers_it_uses(order):
    """Events of the two helper streams: none, and so no stream, where nothing is forked onto it."""
    for nb in range(1, 513):
        first = order.first_step(nb)
        rests = sum(1 for k in range(first) if k % 4 == 3)  # wide updates, one behind each outer block
        batches = sum(1 for k in range(nb) if k % 4 == 3 and k + 2 < nb)  # merges beside the chain; the last are not
        assert (order.rests(nb), order.tri_batches(nb)) == (rests, batches), nb
    assert [order.rests(nb) for nb in (9, 32, 33)] == [0, 0, 3]
    assert [order.tri_batches(nb) for nb in (1, 5, 6, 9, 10)] == [0, 0, 1, 1, 2]


# --------------------------------------------------------------------------- row solver
def test_rows_to_a_workgroup_of_the_small_solver(tmp_path_factory):
    """Five only where sixteen rows per compute unit leave some for a second round and twenty do not; four where all rows
    have 64 unknowns."""
    L = _compile(tmp_path_factory, "solve_plan", """
#include "solve_plan.h"
extern "C" int rows(int64_t c, int all_full) { return thanos::solve_rows_per_group(c, all_full != 0); }
""")
    L.rows.argtypes = [ctypes.c_int64, ctypes.c_int]
    assert [L.rows(c, 0) for c in (1, 4096, 4097, 5120, 5121, 8192, 8193, 10240, 1 << 20)] == [4, 4, 5, 5, 4, 4, 4, 4, 4]
    assert all(L.rows(c, 1) == 4 for c in (1, 4096, 4097, 5120, 5121, 1 << 20))
