"""CPU-side checks of the HIP library: it loads, exports every entry point the
header declares, and its host-side sign rules agree with the oracle's
operator application.  No GPU computation happens here."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

import oracle
import paper_2606_26760_amd as hq
import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    src = open(os.path.join(ROOT, "include", "hinqs.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(hinqs_[a-z0-9_]+)\s*\(", src)))


def test_library_exports_every_declared_symbol():
    lib = hq.load_library()
    names = _declared_symbols()
    assert len(names) >= 14
    for name in names:
        assert hasattr(lib, name), name
    assert set(names) == set(hq.EXPORTED)


def test_opts_defaults_match_header():
    import ctypes
    o = hq.Opts()
    hq.load_library().hinqs_opts_default(ctypes.byref(o))
    assert (o.block, o.max_space, o.max_iter, o.tol, o.precision) == (8, 48, 200, 1e-8, 0)
    assert o.precond_floor == 1e-8 and o.mixed_switch == 1e-5 and o.flags == 0


@pytest.mark.parametrize("norb,na,nb", [(4, 2, 2), (5, 3, 2), (6, 3, 3), (6, 1, 4)])
def test_pair_descriptors_match_oracle(norb, na, nb):
    """Class, holes, particles and sign of every coupled pair of a full space,
    from the library's masked-popcount rules, equal the oracle's
    operator-string signs."""
    rng = np.random.default_rng(norb * 100 + na * 10 + nb)
    alpha, beta = W.full_space(norb, na, nb)
    h = np.eye(norb)
    eri = np.zeros((norb,) * 4)
    o = oracle.Oracle(norb, na, nb, h, eri, 0.0, alpha, beta)
    rows = rng.choice(len(alpha), size=min(len(alpha), 60), replace=False)
    r = o.rows(rows)
    n = 0
    for t, i in enumerate(r["rows"]):
        for e in range(r["rowptr"][t] + 1, r["rowptr"][t + 1]):
            j = int(r["col"][e])
            d = hq.pair_descriptor(int(alpha[i]), int(beta[i]), int(alpha[j]), int(beta[j]))
            typ, neg, h1, h2, p1, p2 = (int(v) for v in hq.decode_descriptor(d))
            et = int(r["etype"][e])
            orb = [int(v) for v in r["orb"][e]]
            assert typ == et
            assert (h1, p1) == (orb[0], orb[2])
            if et >= 3:
                assert (h2, p2) == (orb[1], orb[3])
            assert (-1 if neg else 1) == int(r["sign"][e])
            n += 1
    assert n > 0
    # pairs further apart or identical are not couplings
    assert hq.pair_descriptor(int(alpha[0]), int(beta[0]), int(alpha[0]), int(beta[0])) == 0


def test_binding_refuses_without_gpu():
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is visible")
    with pytest.raises(RuntimeError):
        hq.Hinqs()


def test_create_rejects_half_an_allocator():
    # alloc_fn without free_fn (or the reverse) is refused before any device call
    lib = hq.load_library()
    h = ctypes.c_void_p()
    alloc = hq.ALLOC_FN(lambda n, s, u: None)
    free = hq.FREE_FN(lambda p, s, u: None)
    assert lib.hinqs_create(ctypes.byref(h), 0, None, alloc, hq.FREE_FN(), None) == -1
    assert lib.hinqs_create(ctypes.byref(h), 0, None, hq.ALLOC_FN(), free, None) == -1
    assert h.value is None


_LOOPS = r"""
#include <cstdio>
#include <cstdint>
#include <cstring>
#include <vector>
#include "host_loops.hpp"
using namespace hinqs;
static uint64_t seed = 12345;
static double draw() {
    seed = seed * 6364136223846793005ull + 1442695040888963407ull;
    return (double)(int64_t)(seed >> 11) / 4503599627370496.0 - 1.0;
}
static std::vector<double> fill(size_t n) {
    std::vector<double> v(n);
    for (auto &x : v) x = draw();
    return v;
}
static void show(const std::vector<double> &v) {
    uint64_t h = 1469598103934665603ull;
    for (double x : v) {
        uint64_t b;
        std::memcpy(&b, &x, 8);
        h = (h ^ b) * 1099511628211ull;
    }
    std::printf("%016llx\n", (unsigned long long)h);
}
int main() {
    for (int n : {1, 2, 3, 7, 8, 9, 17, 48}) {
        auto a = fill((size_t)n * n), x = fill(n), y = fill(n), p = fill(n), z = fill((size_t)n * 8), t = fill(8);
        rows_combine(n, n, a.data(), n, x.data(), p.data());
        show(p);
        rank2_update(n, a.data(), n, x.data(), y.data());
        show(a);
        reflect(n, 8, 0.7, x.data(), z.data(), t.data());
        rotate_pair(n, 0.6, 0.8, x.data(), y.data());
        show(z);
        show(x);
        show(y);
    }
}
"""


def test_host_eigensolver_loops_round_alike_on_every_processor(tmp_path):
    """The loops are built for several processors and chosen when the library is loaded: the
    builds that this processor runs give the same bits, so a solve does not depend on the
    host.  Compiled here one by one, with the library's compiler."""
    flags = open("/proc/cpuinfo").read().split()
    src = tmp_path / "loops.cpp"
    src.write_text(_LOOPS)
    hashes = {}
    for name, need, target in (("default", None, ""), ("arch=haswell", "fma", "arch=haswell"),
                               ("avx512f", "avx512f", "avx512f")):
        if need and need not in flags:
            continue
        wide = f'-DHINQS_WIDE=__attribute__((target("{target}")))' if target else "-DHINQS_WIDE="
        exe = tmp_path / f"loops_{len(hashes)}"
        subprocess.run(["/opt/rocm/llvm/bin/clang++", "-O3", "-std=c++17", "-ffp-contract=fast", wide, "-I",
                        os.path.join(ROOT, "paper_2606_26760_amd", "csrc"), str(src), "-o", str(exe)], check=True)
        hashes[name] = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout
    assert len(hashes["default"].split()) == 40
    assert len(hashes) >= 2 and len(set(hashes.values())) == 1, hashes
