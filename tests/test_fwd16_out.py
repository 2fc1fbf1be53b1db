"""The bf16 table forward's output factors (paper_2202_00441_amd/csrc/fwd16_out.h),
on the CPU: the header is compiled into a small program that prints each
activation's range and entries, the kernel's arithmetic on them is emulated
for every bf16 pattern, and the outputs are compared with the oracle's.  The
rule that admits a table (holds) is compared with the oracle's indices: where
it admits one, every pattern has the index of the entry that stands for it."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle as O
from parity import OACT

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ACTS = ["gelu", "silu", "sigmoid", "tanh", "relu", "selu", "softplus"]
PATS = np.arange(1 << 16, dtype=np.uint32).astype(np.uint16)

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "fwd16_out.h"
using namespace fwd16_out;
int main(int argc, char** argv) {
  const int act = std::atoi(argv[1]);
  if (argc > 2) {                     // holds: symmetric flag, then boundaries
    float s[15];
    for (int i = 3; i < argc; ++i) s[i - 3] = std::strtof(argv[i], nullptr);
    std::printf("%d\n", holds(act, std::atoi(argv[2]) != 0, s, argc - 3) ? 1 : 0);
    return 0;
  }
  std::printf("%u %u\n", base_of(act), count_of(act));
  for (int neg = 0; neg < 2 && act != FEWBIT_RELU; ++neg)
    for (uint32_t m = 0; m < count_of(act); ++m) std::printf("%u\n", entry(act, neg != 0, m));
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("fwd16_out")
    src, exe = str(d / "p.cpp"), str(d / "p")
    with open(src, "w") as fh:
        fh.write(PROGRAM)
    # -O2 only: the entries are evaluated at run time here
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2202_00441_amd", "csrc"),
                        src, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def _table(exe, act):
    out = subprocess.run([exe, str(OACT[act])], capture_output=True, text=True, check=True).stdout.split()
    return int(out[0]), int(out[1]), np.array([int(v) for v in out[2:]], dtype=np.uint32)


def _entry_of(base, count):
    """Entry of every pattern: sign (with -0 on the side of +0), magnitude in range."""
    mag = (PATS & 0x7FFF).astype(np.int64)
    m = np.clip(mag - base, 0, count - 1)
    return m + np.where(PATS > 0x8000, count, 0)


def _value(pats):
    return (pats.astype(np.uint32) << 16).view(np.float32)


@pytest.mark.parametrize("act", [a for a in ACTS if a != "relu"])
def test_outputs_are_correctly_rounded(program, act):
    base, count, entries = _table(program, act)
    assert entries.size == 2 * count and not (entries & 15).any()
    top = _value(np.array([base + count - 1], np.uint16))[0]
    x = _value(PATS)
    y_ref = O.fwd(OACT[act], O.BF16, 1, np.float32([1.0]), PATS)[0]
    ok = (PATS & 0x7FFF) <= 0x7F80                      # NaNs have no entry of their own
    for code in (0, 1, 8, 15):
        word = entries[_entry_of(base, count)] | np.uint32(0 if act in ("gelu", "silu") else code)
        t = word.view(np.float32)
        with np.errstate(all="ignore"):
            if act == "softplus":
                y = np.where(x > 0, x, np.float32(0)) + t
            elif act == "sigmoid":
                y = t
            elif act == "tanh":
                y = np.clip(x, -top, top) * t
            else:
                y = np.maximum(x, -top) * t
        got = O.round_array(O.BF16, y[ok].astype(np.float64))
        same = (got == y_ref[ok]) | (((got | y_ref[ok]) & 0x7FFF) == 0)
        assert same.all(), (act, code, PATS[ok][~same][:8], got[~same][:8], y_ref[ok][~same][:8])


@pytest.mark.parametrize("act", ACTS)
def test_admitted_boundaries_have_one_index_per_entry(program, act):
    base, count, _ = _table(program, act)
    lo, hi = _value(np.array([base, base + count - 1], np.uint16))
    below, above = np.nextafter(lo, np.float32(0)), np.nextafter(lo, np.float32(1))
    edges = [0.0, -0.0, 1e-40, -1e-40, lo, -lo, below, -below, above, -above, 0.5, -0.5, 3.0,
             np.nextafter(hi, np.float32(0)), -np.nextafter(hi, np.float32(0)), hi, -hi, 2 * hi, -2 * hi]
    entry = _entry_of(base, count)
    finite = (PATS & 0x7FFF) <= 0x7F80
    rng = np.random.default_rng(5)
    admitted = 0
    for trial in range(60):
        sym = trial % 3 == 2
        k = 1 if trial < len(edges) else 3
        s = [edges[trial]] if k == 1 else list(rng.choice(edges, 3, replace=False))
        s = np.unique(np.float32(s))
        if s.size != k:
            continue
        args = [program, str(OACT[act]), str(int(sym))] + [repr(float(v)) for v in s]
        if subprocess.run(args, capture_output=True, text=True, check=True).stdout.strip() != "1":
            continue
        admitted += 1
        _, _, idx = O.fwd(OACT[act], O.BF16, 1 if k == 1 else 2, s, PATS, symmetric=sym, want_idx=True)
        idx = np.asarray(idx).astype(np.int64)
        for e in np.unique(entry):
            of_entry = idx[(entry == e) & finite]
            assert (of_entry == of_entry[0]).all(), (act, sym, s, int(e))
    assert admitted >= 4
