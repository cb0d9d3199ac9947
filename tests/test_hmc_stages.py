"""The stages of the trajectory integrators (csrc/hmc_stages.h, host code) on the CPU: the
sequence of each integrator written out, and trajectories of the longest step counts, whose
stages take no list."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2302_00850_amd", "csrc")
LAMBDA = 0.1931833275037836

PROBE = r"""
#include "hmc_stages.h"
using namespace cola;
static cola_hmc_params_t params(int integrator, double eps, int nsteps, int n_gauge) {
    cola_hmc_params_t p{};
    p.integrator = integrator, p.eps = eps, p.nsteps = nsteps, p.n_gauge = n_gauge;
    return p;
}
extern "C" long long probe_count(int integrator, double eps, int nsteps, int n_gauge) {
    return stage_count(params(integrator, eps, nsteps, n_gauge));
}
extern "C" void probe_at(int integrator, double eps, int nsteps, int n_gauge, long long k,
                         double *o) {
    const Stage s = stage_at(params(integrator, eps, nsteps, n_gauge), k);
    o[0] = s.fermions, o[1] = s.eps_f, o[2] = s.eps_g, o[3] = s.eps_u;
}
"""


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    d = tmp_path_factory.mktemp("stages")
    src, so = str(d / "probe.cpp"), str(d / "probe.so")
    with open(src, "w") as f:
        f.write(PROBE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", so],
                   check=True)
    lib = ctypes.CDLL(so)
    lib.probe_count.restype = ctypes.c_longlong
    lib.probe_count.argtypes = [ctypes.c_int, ctypes.c_double, ctypes.c_int, ctypes.c_int]
    lib.probe_at.argtypes = lib.probe_count.argtypes + [ctypes.c_longlong,
                                                        ctypes.POINTER(ctypes.c_double)]
    return lib


def _at(probe, integrator, eps, nsteps, n_gauge, k):
    o = (ctypes.c_double * 4)()
    probe.probe_at(integrator, eps, nsteps, n_gauge, k, o)
    return tuple(o)


def _written_out(integrator, eps, n, m):
    """(fermion kick, its step, gauge kick's step) up to the next link update, and that
    update's step: the kicks and updates of each integrator one after the other, adjoining
    ones of the same kind added."""
    v = []
    if integrator == 0:
        for k in range(n + 1):
            e = 0.5 * eps if k in (0, n) else eps
            v.append((1, e, e, eps))
    elif integrator == 1:
        v.append((1, LAMBDA * eps, LAMBDA * eps, 0.5 * eps))
        for k in range(n):
            mid, e = (1 - 2 * LAMBDA) * eps, (LAMBDA if k == n - 1 else 2 * LAMBDA) * eps
            v += [(1, mid, mid, 0.5 * eps), (1, e, e, 0.5 * eps)]
    else:
        hs = eps / m
        for k in range(n + 1):
            end = k in (0, n)
            v.append((1, 0.5 * eps if end else eps, 0.5 * hs if end else hs, hs))
            if k < n:
                v += [(0, 0.0, hs, hs)] * (m - 1)
    return v


@pytest.mark.parametrize("integrator,n_gauge", [(0, 1), (1, 1), (2, 1), (2, 2), (2, 5)])
@pytest.mark.parametrize("nsteps", [1, 2, 3, 20])
def test_sequence(probe, integrator, n_gauge, nsteps):
    eps = 0.07
    want = _written_out(integrator, eps, nsteps, n_gauge)
    assert probe.probe_count(integrator, eps, nsteps, n_gauge) == len(want)
    for k, w in enumerate(want):
        assert _at(probe, integrator, eps, nsteps, n_gauge, k) == pytest.approx(w, rel=1e-15)


def test_longest_trajectories(probe):
    n = 2**31 - 1
    for integrator, m, count in ((0, 1, n + 1), (1, 1, 2 * n + 1), (2, n, n * n + 1)):
        assert probe.probe_count(integrator, 0.5, n, m) == count
        first = _at(probe, integrator, 0.5, n, m, 0)
        assert first == _at(probe, integrator, 0.5, n, m, count - 1) and first[0] == 1
        assert first != _at(probe, integrator, 0.5, n, m, count - 2)
