"""The library's rules for kernel variants and splits of the work (csrc/gt_shape.hpp), compiled for the CPU: tests
ask them which variant a call takes, so that a change of a rule cannot empty a test unnoticed."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

SIMDS = 1024                                       # of an MI355X: 256 compute units of four
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2305_00645_amd", "csrc")
SOURCE = r"""
#include "gt_shape.hpp"
extern "C" void infer(u64 simds, u32 lgi, u64 ngrp, u32 ntrees, u32 H, u32 d, int thr, u32 *out)
{
    const InferShape s = infer_shape(simds, lgi, ngrp, ntrees, H, d, thr != 0);
    out[0] = s.nq; out[1] = s.nw; out[2] = s.noct;
}
extern "C" void grid(u64 simds, int mode, int ndot, int sums, u32 w, u64 N8, u64 *out)
{
    const GridShape s = grid_shape(simds, mode, ndot, sums != 0, w, N8);
    out[0] = s.ntile; out[1] = s.nkc; out[2] = s.kchunk; out[3] = s.alone; out[4] = s.rps; out[5] = s.waves;
}
extern "C" int staged(u32 noct, int thr) { return staged_sums(noct, thr != 0); }
extern "C" int bytes(u64 simds, u64 np, u64 d) { return onehot_bytes(simds, np, d); }
extern "C" int early(u64 n, u64 tile_bytes) { return split_early(n, tile_bytes); }
extern "C" int pairs(u64 simds, u64 n) { return eq_pairs(simds, n); }
extern "C" int comps(u32 H, u64 ncol) { return tile_rows(H, ncol).comps; }
extern "C" void xy(u64 simds, u64 N8, u32 d, u32 K, u64 *out)
{
    const XySplit s = xy_split(simds, N8, d, K);
    out[0] = s.tk; out[1] = s.items; out[2] = s.groups;
}
extern "C" int few(int xcols, u64 nh, u64 nblk, u64 ncol) { return count_few(xcols != 0, nh, nblk, ncol); }
"""
STORE, COMMON, ROWS = 0, 1, 2                      # modes of the equality grid


@functools.lru_cache(None)
def _lib():
    with tempfile.TemporaryDirectory() as tmp:
        src, so = os.path.join(tmp, "shapes.cpp"), os.path.join(tmp, "shapes.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, "-o", so, src], check=True)
        L = C.CDLL(so)
    u32, u64, i, vp = C.c_uint32, C.c_uint64, C.c_int, C.c_void_p
    L.infer.argtypes, L.infer.restype = [u64, u32, u64, u32, u32, u32, i, vp], None
    L.grid.argtypes, L.grid.restype = [u64, i, i, i, u32, u64, vp], None
    L.staged.argtypes, L.staged.restype = [u32, i], i
    L.bytes.argtypes, L.bytes.restype = [u64, u64, u64], i
    L.early.argtypes, L.early.restype = [u64, u64], i
    L.pairs.argtypes, L.pairs.restype = [u64, u64], i
    L.comps.argtypes, L.comps.restype = [u32, u64], i
    L.xy.argtypes, L.xy.restype = [u64, u64, u32, u32, vp], None
    L.few.argtypes, L.few.restype = [i, u64, u64, u64], i
    return L


def infer(NI, H, d, thr, tile=0, ntrees=1):
    """(kernel, groups of 8 instances per workgroup) of an inference; tile: instances per workgroup asked for, 0: none."""
    out = (C.c_uint32 * 3)()
    _lib().infer(SIMDS, tile.bit_length() - 1 if tile else 0, (NI + 7) // 8, ntrees, H, d, int(thr), out)
    nq, nw, noct = out
    return ("ahead%d" % nq if nq else "infer%d" % nw), noct


def staged(noct, thr):
    """Whether single wavefronts with that many groups add up their sums through LDS."""
    return bool(_lib().staged(noct, int(thr)))


def grid(mode, w, N, sums=1, tile_sums=False):
    """dict(tiles, ranges, columns, alone, adjacent, waves) of an equality grid of N rows and w columns; sums: inner products;
    tile_sums: the leaf one-hot is written with its sums."""
    out = (C.c_uint64 * 6)()
    _lib().grid(SIMDS, mode, sums, int(tile_sums), w, (N + 7) // 8 * 8, out)
    return dict(tiles=out[0], ranges=out[1], columns=out[2], alone=bool(out[3]), adjacent=out[4], waves=out[5])


def onehot_bytes(nodes, d):
    """Whether a partition by products after a level of that many nodes writes its one-hot as bytes in the launch that tests."""
    return bool(_lib().bytes(SIMDS, nodes, d))


def split_early(nodes, N, ncol, planes=3):
    """Whether a level's node split loads its words before the block function; planes: of the columns' tiles, 6 where they are kept per party."""
    return bool(_lib().early(nodes * ncol, planes * ((ncol + 63) // 64 * 64 + 64) * ((N + 31) // 32) * 256))


def eq_pairs(n):
    """Whether equality tests of n elements take tiles of 40, two per lane."""
    return bool(_lib().pairs(SIMDS, n))


def setup(N, d, K, H):
    """dict(comps, features, items, groups) of a training's set-up: the columns kept once per component, features of a workgroup's part, blocks x
    parts, workgroups."""
    out = (C.c_uint64 * 3)()
    _lib().xy(SIMDS, (N + 7) // 8 * 8, d, K, out)
    return dict(comps=bool(_lib().comps(H, d * K + K)), features=out[0], items=out[1], groups=out[2])


def few(nodes, N, ncol):
    """Whether a level of that many nodes counts all its columns on the narrow tiles, where the columns are stored once."""
    return bool(_lib().few(1, nodes, (N + 31) // 32, ncol))
