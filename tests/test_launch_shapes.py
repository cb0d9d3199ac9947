"""The launch-shape rules (csrc/shapes.h, host code) on the CPU, over lattices from 2^4 to
48^3 x 96, every precision and right-hand-side count: each default is a shape the kernels
accept, and what the rules say of it holds."""
import ctypes
import itertools
import os
import subprocess
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2302_00850_amd", "csrc")

PROBE = r"""
#include <cstring>
#include "shapes.h"
using namespace cola;
static void put(const TuneEntry &t, int *o) {
    const int v[7] = {t.rpt, t.sites_per_block, t.grid, t.tchunk, t.tile_y, t.tile_z, t.stage};
    memcpy(o, v, sizeof v);
}
extern "C" {
void probe_default(const int *d, int prec, int nrhs, int both, int clover, int *o) {
    put(default_entry(make_geom(d), prec, nrhs, both, clover), o);
}
void probe_plain(const int *d, int prec, int nrhs, int both, int clover, int *o) {
    put(plain_entry(make_geom(d), prec, nrhs, both, clover), o);
}
void probe_flic(const int *d, int prec, int nrhs, int both, int *o) {
    put(flic_entry(make_geom(d), prec, nrhs, both), o);
}
int probe_candidates(const int *d, int prec, int nrhs, int both, int clover, int *o, int most) {
    const auto c = tune_candidates(make_geom(d), prec, nrhs, both, clover);
    for (int k = 0; k < (int)c.size() && k < most; ++k) put(c[k], o + 7 * k);
    return (int)c.size();
}
int probe_key(const char *arch, int num_cu, const char *key, char *o, int most) {
    const std::string s = table_key(arch, num_cu, key);
    strncpy(o, s.c_str(), most - 1);
    return (int)s.size();
}
void probe_tile(const int *d, int most, int *o) { best_tile(make_geom(d), most, o, o + 1); }
int probe_valid(const int *d, int prec, int nrhs, const int *s) {
    TuneEntry t;
    t.rpt = s[0], t.sites_per_block = s[1], t.grid = s[2], t.tchunk = s[3];
    t.tile_y = s[4], t.tile_z = s[5], t.stage = s[6];
    const Geom g = make_geom(d);
    return shape_valid(g, prec, nrhs, t) && (t.stage != 1 || stage_ok(g, prec, nrhs, t));
}
}
"""

LATTICES = [(2, 2, 2, 2), (4, 4, 4, 4), (6, 4, 4, 10), (20, 18, 14, 30), (16, 16, 16, 32),
            (2, 46, 34, 8), (24, 24, 24, 48), (32, 32, 32, 64), (48, 48, 48, 96)]
FP64, FP64_12, FP32, FP16 = range(4)
KINDS = list(itertools.product(LATTICES, (FP64, FP64_12, FP32, FP16), range(1, 17), (0, 1)))


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    d = tmp_path_factory.mktemp("shapes")
    src, so = str(d / "probe.cpp"), str(d / "probe.so")
    with open(src, "w") as f:
        f.write(PROBE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", so],
                   check=True)
    return ctypes.CDLL(so)


def _dims(d):
    return (ctypes.c_int * 4)(*d)


def _shape(fn, *args):
    out = (ctypes.c_int * 7)()
    fn(*args, out)
    return tuple(out)


def test_defaults_are_accepted(probe):
    for d, prec, nrhs, both in KINDS:
        for clover in (0, 1):
            s = _shape(probe.probe_default, _dims(d), prec, nrhs, both, clover)
            assert probe.probe_valid(_dims(d), prec, nrhs, (ctypes.c_int * 7)(*s)), \
                (d, prec, nrhs, both, clover, s)
            s = _shape(probe.probe_plain, _dims(d), prec, nrhs, both, clover)
            assert s[6] != 2 and probe.probe_valid(_dims(d), prec, nrhs, (ctypes.c_int * 7)(*s))


def test_flic_defaults_are_shapes_of_the_flic_kernel(probe):
    """One rhs per lane, links neither staged nor split over wavefronts, and a block of at
    most 256 lanes with that."""
    for d, prec, nrhs, both in KINDS:
        if prec == FP16:
            continue
        s = _shape(probe.probe_flic, _dims(d), prec, nrhs, both)
        assert s[0] == 1 and s[6] == 0 and s[1] * nrhs <= 256, (d, prec, nrhs, both, s)
        assert probe.probe_valid(_dims(d), prec, nrhs, (ctypes.c_int * 7)(*s))


def test_tuner_times_the_defaults(probe):
    """The default shape and the one-lane-per-(site, rhs) default are among the candidates, so
    tuning cannot settle on a slower one; every candidate is a shape the kernels accept, and
    none is timed twice."""
    buf = (ctypes.c_int * (7 * 4096))()
    for d, prec, nrhs, both in KINDS:
        for clover in (0, 1):
            n = probe.probe_candidates(_dims(d), prec, nrhs, both, clover, buf, 4096)
            assert 0 < n <= 4096
            cand = [tuple(buf[7 * k:7 * k + 7]) for k in range(n)]
            assert len(set(cand)) == n
            assert _shape(probe.probe_default, _dims(d), prec, nrhs, both, clover) in cand
            assert _shape(probe.probe_plain, _dims(d), prec, nrhs, both, clover) in cand
            for s in cand:
                assert probe.probe_valid(_dims(d), prec, nrhs, (ctypes.c_int * 7)(*s)), s


def test_tables_of_earlier_kernels_are_not_used(probe):
    """A line of a table written before the kernels and defaults changed (device, key, shape;
    no version) does not answer a launch of today's library, and the keys still tell devices
    and launches apart."""
    def key(arch, cu, k):
        buf = ctypes.create_string_buffer(256)
        n = probe.probe_key(arch, cu, k, buf, 256)
        assert n < 256
        return buf.value
    hop = b"hop:16x16x16x32:p2:r1:e1:n1"
    line = b"gfx950:256 " + hop + b" 1 128 0 1 0 0 0 0.020000"
    now = key(b"gfx950", 256, hop)
    assert b" ".join(line.split()[:2]) != now
    # what the file holds of it is read back as two words (of up to 127 and 159 bytes)
    assert len(now.split()) == 2 and now.split()[1] == hop and len(now.split()[0]) < 128
    others = [key(b"gfx950", 304, hop), key(b"gfx942", 256, hop), key(b"gfx950", 256, hop + b":b")]
    assert len({now, *others}) == 4


def test_links_are_staged_from_the_stated_rhs_count(probe):
    """FP32 and FP16 launches with one lane per (site, rhs) stage links from five rhs on, and
    with four where no clover block is read and the launch keeps at least 1024 blocks; never
    with fewer."""
    for d, prec, nrhs, both in KINDS:
        blocks = d[0] * d[1] * d[2] * d[3] // 2 * (2 if both else 1) / 32
        for clover in (0, 1):
            staged = _shape(probe.probe_plain, _dims(d), prec, nrhs, both, clover)[6] == 1
            want = prec in (FP32, FP16) and (
                nrhs >= 5 or (nrhs == 4 and not clover and blocks >= 2048))
            assert staged == want, (d, prec, nrhs, both, clover)


# (lattice, precision, both parities, clover): the kernel that was faster; one rhs, then rhs
FASTER = [
    ((16, 16, 16, 32), FP32, 1, 1, "directions"), ((18, 18, 18, 30), FP32, 1, 1, "sites"),
    ((20, 20, 20, 32), FP32, 1, 1, "sites"), ((16, 16, 16, 32), FP64_12, 1, 1, "directions"),
    ((20, 20, 20, 24), FP64_12, 1, 1, "sites"), ((20, 20, 20, 32), FP64_12, 1, 1, "sites"),
    ((20, 20, 20, 32), FP64, 1, 1, "directions"), ((24, 24, 24, 32), FP64, 1, 1, "sites"),
    ((24, 24, 24, 32), FP32, 0, 1, "directions"), ((20, 20, 20, 32), FP64, 0, 1, "directions"),
    ((20, 20, 20, 32), FP64_12, 0, 1, "directions"), ((24, 24, 24, 32), FP64, 0, 1, "sites"),
    ((28, 28, 28, 48), FP64_12, 1, 0, "directions"), ((28, 28, 28, 48), FP64, 1, 0, "directions"),
    ((24, 24, 24, 32), FP64_12, 0, 0, "directions"), ((28, 28, 28, 48), FP64, 0, 0, "sites"),
    ((32, 32, 32, 64), FP32, 0, 0, "sites"), ((32, 32, 32, 64), FP64, 1, 0, "sites"),
]


FASTER = [c[:4] + (1, c[4]) for c in FASTER] + [
    ((12, 12, 12, 8), FP32, 1, 1, 8, "sites"), ((8, 8, 8, 16), FP32, 1, 1, 12, "sites"),
    ((8, 8, 8, 16), FP32, 1, 1, 8, "directions"), ((12, 12, 12, 24), FP32, 1, 1, 3, "directions"),
    ((8, 8, 8, 16), FP64, 1, 1, 12, "sites"), ((12, 12, 12, 12), FP64, 1, 1, 5, "directions"),
    ((16, 16, 16, 16), FP64, 1, 1, 3, "sites"), ((16, 16, 16, 16), FP64_12, 0, 1, 3, "sites"),
    ((12, 12, 12, 24), FP64, 0, 1, 5, "directions"), ((12, 12, 12, 12), FP64, 1, 0, 12, "directions"),
    ((12, 12, 12, 16), FP64, 1, 1, 7, "directions"), ((12, 12, 12, 8), FP64, 1, 1, 16, "directions"),
    ((20, 18, 14, 30), FP64_12, 1, 1, 1, "directions"),
]


@pytest.mark.parametrize("lattice,prec,both,clover,nrhs,faster", FASTER)
def test_default_is_the_kernel_measured_faster(probe, lattice, prec, both, clover, nrhs, faster):
    s = _shape(probe.probe_default, _dims(lattice), prec, nrhs, both, clover)
    assert (s[6] == 2) == (faster == "directions")


def _best_tile(d, most):
    """The largest tile of `most` sites by trying every pair of extents."""
    best = (0, 0)
    for y in range(2, d[1] + 1):
        for z in range(2, d[2] + 1):
            if d[1] % y or d[2] % z or d[0] // 2 * y * z > most:
                continue
            if y * z > best[0] * best[1] or (
                    y * z == best[0] * best[1] and abs(y - z) < abs(best[0] - best[1])):
                best = (y, z)
    return best


def test_tile_search(probe):
    """The search finds the tile that trying every pair finds, and where the extents are large
    it does not cost a launch's time: it runs on every call that has no tuned shape.  All
    pairs of 512 x 512 take 190 us, the divisors among them 5."""
    out = (ctypes.c_int * 2)()
    for d in LATTICES + [(2, 512, 96, 2), (4, 30, 210, 4), (6, 22, 26, 2)]:
        for most in (0, 1, 4, 64, 288, 900, 1024, 2048, 4096, 8192):
            probe.probe_tile(_dims(d), most, out)
            assert tuple(out) == _best_tile(d, most), (d, most)
    d, took = _dims((2, 512, 512, 2)), []
    for _ in range(20):
        t0 = time.perf_counter()
        probe.probe_tile(d, 8192, out)
        took.append(time.perf_counter() - t0)
    assert min(took) < 60e-6


def test_flic_blocks(probe):
    """FLIC launches of several rhs: a block is one wavefront where the rhs fill it, and no
    launch leaves most compute units without a block while its blocks are of several
    wavefronts."""
    for d, prec, nrhs, both in KINDS:
        if prec == FP16 or nrhs == 1:
            continue
        _, T, _, tchunk, *_ = _shape(probe.probe_flic, _dims(d), prec, nrhs, both)
        sites = d[0] * d[1] * d[2] * d[3] // 2 * (2 if both else 1)
        if nrhs in (2, 4, 8, 16):
            assert T * nrhs == 64, (d, prec, nrhs, both)
        assert T * nrhs <= 64 or sites / tchunk / T >= 200 or T * nrhs < 128, (d, prec, nrhs, both)


def test_tiles_cut_the_timeslice_only_where_it_is_large(probe):
    """A tile is never the whole timeslice (the plain order is the same and cheaper), and with
    several rhs a timeslice of up to 1.25 times the tile size stays whole: 20 x 18 x 14 has
    2520 sites of a parity."""
    for d, prec, nrhs, both in KINDS:
        for fn, more in ((probe.probe_plain, (0,)), (probe.probe_flic, ())):
            s = _shape(fn, _dims(d), prec, nrhs, both, *more)
            assert (s[4], s[5]) != (d[1], d[2])
    for prec, nrhs in ((FP32, 3), (FP32, 12), (FP16, 12), (FP64, 2), (FP64, 3)):
        s = _shape(probe.probe_plain, _dims((20, 18, 14, 30)), prec, nrhs, 0, 0)
        assert s[4:6] == (0, 0)
    assert _shape(probe.probe_plain, _dims((24, 24, 24, 48)), FP32, 12, 0, 0)[4:6] == (12, 12)
