"""The split-key plan on the host: csrc/ism_split_plan.h (built here as plain
C++) with the device side of csrc/ism_plan.h repeated in numpy, so that every
read and write that the plan leads to is checked without a GPU.

The kernels' own shapes are the reference: split_attn_kernel serves 32
columns and steps 32 keys, the forward kernel 128 columns and 64 keys.
"""

import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2408_00539_amd", "csrc")
SHIM = """
#include "ism_split_plan.h"
extern "C" int kind_of(int batch, long total, int rows, int hq, int hkv, int cap) {
  return ism::prefill_kind(batch, total, rows, hq, hkv, cap);
}
extern "C" void plan_of(int kind, int batch, long total, int rows, int hq, int hkv, int d,
                        long max_len, int fixed, int limited, long ws, long *out) {
  const ism::SplitPlan p = ism::split_plan((ism::SplitKind)kind, batch, total, rows, hq, hkv, d,
                                           max_len, fixed, limited, ws);
  const long v[] = {p.colw, p.col_groups, p.col_stride, p.budget, p.max_units, p.max_splits,
                    p.tile_shift, p.min_tiles, p.whole_tiles, (long)p.part_bytes,
                    (long)p.ml_bytes, (long)p.plan_bytes};
  for (int i = 0; i < 12; ++i) out[i] = v[i];
}
"""
ROW_TILES, ROW_TILES_SPLIT, ONE_WAVE, DECODE = 0, 1, 2, 3
COLS = {ROW_TILES_SPLIT: 128, ONE_WAVE: 32, DECODE: 32}
KEYS = {ROW_TILES_SPLIT: 64, ONE_WAVE: 32, DECODE: 32}


class Plan:
    def __init__(self, lib, kind, batch, total, rows, hq, hkv, d, max_len, fixed=0, ws=None):
        out = (ctypes.c_long * 12)()
        lib.plan_of(kind, batch, ctypes.c_long(total), rows, hq, hkv, d, ctypes.c_long(max_len),
                    fixed, ws is not None, ctypes.c_long(ws or 0), out)
        (self.colw, self.col_groups, self.col_stride, self.budget, self.max_units,
         self.max_splits, self.tile_shift, self.min_tiles, self.whole_tiles, self.part_bytes,
         self.ml_bytes, self.plan_bytes) = out
        self.key = tuple(out)
        self.bytes = self.part_bytes + self.ml_bytes + self.plan_bytes


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    if not cxx:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                        "-I" + CSRC, "-o", str(d / "shim.so"), str(d / "shim.cpp")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = ctypes.CDLL(str(d / "shim.so"))
    out.kind_of.argtypes = [ctypes.c_int, ctypes.c_long] + 4 * [ctypes.c_int]
    return out


def units(p, cached, rows, group, cap, fixed=0):
    """(dialogue, chunk, chunks, first tile, tiles, keys, column groups) of
    every unit of one KV head, as the device plan makes them."""
    keys = np.clip(cached.astype(np.int64) + rows, 1, cap)
    t = np.where(rows > 0, ((keys - 1) >> p.tile_shift) + 1, 0)
    g = np.minimum(-(-rows.astype(np.int64) * group // p.colw), p.col_groups)
    def chunks(lc):
        n = np.where(t <= p.whole_tiles, 1, np.minimum(fixed or -(-t // lc), p.max_splits))
        per = np.where(n <= 1, np.maximum(t, 1), -(-t // np.maximum(n, 1)))
        return per, -(-t // per)

    lc = 1
    if not fixed and p.max_splits > 1 and not p.budget:
        lc = p.min_tiles
    elif not fixed and p.max_splits > 1:
        total, longest = np.float32((t * g).sum()), 1 << 26

        groups, lc, count = int(g.sum()), 0, p.colw == 32 and len(rows) <= 256
        room = p.budget - groups * (0 if p.colw != 32 else 0.5 if count else 1)
        while True:
            x = np.float32(total / np.float32(max(room, 1)) * np.float32(1.0001))
            lc = max(int(min(x if room >= 1 else 1e9, longest)) + 1, p.min_tiles,
                     lc + (lc >> 4) + 1 if lc else 0)
            c = int((np.minimum(-(-t // lc), p.max_splits) * g).sum())
            if not count or c <= p.budget or lc > longest:
                break
            room = p.budget - (c - float(total) / lc)
    per, n = chunks(lc)
    out = []
    for b in range(len(rows)):
        out += [(b, i, int(n[b]), i * int(per[b]), int(min(per[b], t[b] - i * per[b])),
                 int(keys[b]), int(g[b])) for i in range(int(n[b]))]
    return out


def check(p, kind, cached, rows, hq, hkv, d, cap, fixed=0):
    group = hq // hkv
    assert (p.colw, 1 << p.tile_shift) == (COLS[kind], KEYS[kind])
    u = units(p, cached, rows, group, cap, fixed)
    # the grid, and the partials that it writes
    assert sum(x[-1] for x in u) <= p.max_units
    if p.max_splits > 1:
        slots = p.max_units * hkv * p.col_stride
        assert p.part_bytes >= slots * d * 4 and p.ml_bytes >= slots * 8
        assert p.plan_bytes >= len(rows) * 8
    for b, i, n, tile0, tiles, keys, g in u:
        # every chunk begins at a key that exists, and the last one ends at the end
        assert tiles > 0 and tile0 * KEYS[kind] < keys <= cap
        assert (i == n - 1) == ((tile0 + tiles) * KEYS[kind] >= keys)
        # the columns of a group fit its slot, and the groups hold every column
        cols = int(rows[b]) * group
        assert g * COLS[kind] >= cols and min(cols, COLS[kind]) <= p.col_stride


HEADS = (1, 2, 3, 8, 31, 32, 33, 40, 64, 127, 128, 129, 160, 256, 320, 4096)


@pytest.mark.parametrize("rows", [1, 2, 3, 8, 32, 33, 100])
def test_prefill_plan_fits_its_kernel(lib, rows):
    """Over new rows and query heads per KV head, dense and ragged."""
    rng = np.random.default_rng(rows)
    kinds = set()
    for group in HEADS:
        for hkv, batch in ((1, 1), (1, 3), (2, 11), (8, 70), (16, 200), (4, 600)):
            for cap in (rows + 63, 1025, 4096, 8192, 200000):
                kind = lib.kind_of(batch, rows * batch, rows, hkv * group, hkv, cap)
                if kind == ROW_TILES:
                    continue
                kinds.add(kind)
                p = Plan(lib, kind, batch, rows * batch, rows, hkv * group, hkv, 128, cap)
                one_long = np.where(np.arange(batch) == batch // 2, cap - rows, cap // 100)
                for cached in (np.full(batch, cap - rows), np.full(batch, max(0, cap // 2 - rows)),
                               rng.integers(0, cap - rows + 1, size=batch), one_long):
                    for new in (np.full(batch, rows), rng.integers(0, rows + 1, size=batch)):
                        check(p, kind, cached, new, hkv * group, hkv, 128, cap)
    assert ROW_TILES_SPLIT in kinds and (rows > 32 or ONE_WAVE in kinds)


DECODES = [(1, 32, 8, 128, 2500), (1, 32, 8, 128, 8192), (9, 8, 2, 128, 3000),
           (9, 40, 1, 64, 3000), (4, 32, 8, 128, 3000), (40, 32, 8, 128, 4000),
           (30, 16, 8, 64, 5000), (3, 64, 1, 128, 130), (200, 64, 8, 128, 900),
           (101, 32, 8, 128, 32001), (256, 8, 4, 64, 4000), (300, 32, 2, 128, 4000),
           (700, 24, 2, 64, 300), (5, 300, 100, 64, 9000)]


@pytest.mark.parametrize("batch,hq,hkv,d,max_len", DECODES)
@pytest.mark.parametrize("fixed", [0, 1, 2, 3, 16, 64])
def test_decode_plan_in_its_workspace(lib, batch, hq, hkv, d, max_len, fixed):
    """With a workspace of the plan's own size it is the plan without a limit;
    smaller ones give plans that fit them."""
    rng = np.random.default_rng(batch + fixed)
    args = (lib, DECODE, batch, batch, 1, hq, hkv, d, max_len, fixed)
    full = Plan(*args)
    assert Plan(*args, ws=full.bytes).key == full.key
    rows = np.ones(batch, dtype=np.int64)
    for ws in [full.bytes * i // 16 // 256 * 256 for i in range(1, 16)] + [256, full.bytes - 256]:
        if ws <= 0:
            continue
        p = Plan(*args, ws=ws)
        assert p.bytes <= ws and p.max_units <= full.max_units
        one_long = np.where(np.arange(batch) == batch // 2, max_len - 1, max_len // 100)
        for cached in (np.full(batch, max_len - 1), rng.integers(0, max_len, size=batch),
                       one_long):
            check(p, DECODE, cached, rows, hq, hkv, d, max_len, fixed)


def test_accepted_noalloc_steps_fit_the_scratch(lib):
    """Every step whose smallest workspace is at most the limit of
    ism_attn_decode_noalloc fits its whole plan into the library's scratch."""
    text = open(os.path.join(CSRC, "ism_api.hip")).read()
    scratch = int(re.search(r"kScratchBytes = (\d+)u << 20", text).group(1)) << 20
    limit, most = 8 << 20, 0
    for d in (64, 128):
        for group in HEADS:
            for hkv in (1, 2, 8, 32, 100, 256):
                hq = group * hkv
                if hq > 8192:
                    continue
                top = limit // (hq * (d + 2) * 4)
                for batch in {1, 2, 3, 17, top // 3, top}:
                    for fixed in (0, 1, 2, 64):
                        # the smallest workspace holds at least this
                        if batch < 1 or batch * hq * max(fixed, 1) * (d + 2) * 4 > limit:
                            continue
                        for max_len in (1, 700, 8192, 1 << 20):
                            p = Plan(lib, DECODE, batch, batch, 1, hq, hkv, d, max_len, fixed)
                            most = max(most, p.bytes)
                            assert p.bytes <= scratch, (batch, hq, hkv, d, fixed, max_len)
    assert most > limit


@pytest.mark.parametrize("batch,hkv,d", [(100, 8, 128), (64, 8, 128), (30, 8, 64), (127, 8, 128)])
def test_equal_decodes_fill_their_grid(lib, batch, hkv, d):
    """A step of equal dialogues launches no more workgroups than the chip
    holds at once, and as many chunks as the grid has room for."""
    rows = np.ones(batch, dtype=np.int64)
    for keys in (900, 4001, 8193):
        p = Plan(lib, DECODE, batch, batch, 1, 4 * hkv, hkv, d, keys)
        assert p.max_units * hkv <= 1024
        chunks = len(units(p, np.full(batch, keys - 1), rows, 4, keys)) // batch
        most = min(p.max_units // batch, -(-keys // 128))
        # (chunks of whole tiles: evening them out can drop some)
        assert most == 1 and chunks == 1 or chunks > 0.7 * most


def test_one_long_dialogue_among_many(lib):
    """Drafted rows: a dialogue that decides the call is cut, also where whole
    dialogues alone fill the chip; caches with no room for one need no plan."""
    cached = np.array([32000] + [300] * 255)
    rows = np.full(256, 8, dtype=np.int64)
    p = Plan(lib, ONE_WAVE, 256, 2048, 8, 32, 8, 128, 32768)
    u = units(p, cached, rows, 4, 32768)
    assert max(x[4] for x in u) * KEYS[ONE_WAVE] < 4096
    assert Plan(lib, ONE_WAVE, 256, 2048, 8, 32, 8, 128, 4096).max_splits == 1


def test_short_rows_stay_whole(lib):
    """Row-tiled segments over short caches, or short dialogues in long ones,
    are not cut."""
    assert lib.kind_of(1, 200, 200, 32, 8, 1024) == ROW_TILES
    assert lib.kind_of(1, 200, 200, 32, 8, 1088) == ROW_TILES_SPLIT
    p = Plan(lib, ROW_TILES_SPLIT, 3, 120, 40, 32, 8, 128, 8192)
    u = units(p, np.array([300, 472, 2000]), np.full(3, 40), 4, 8192)
    assert [x[2] for x in u][:2] == [1, 1] and u[2][2] > 1
