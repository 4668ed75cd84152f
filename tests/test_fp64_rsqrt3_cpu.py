"""q^(-3/2) of the FP64 pair sum (gccd_fp64.h, rsqrt3_pos), built for the host
(the estimate from single precision in place of the hardware's, then the same
correction), against 40-digit references over the squared distances it meets
(softening 1 nm to centimetres): at most 1.5 units in the last place, and a
smaller rms error than 1/(q sqrt q) in IEEE double arithmetic."""
import os
import subprocess

import numpy as np
import pytest

mp = pytest.importorskip("mpmath")

INC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2203_11043_amd", "csrc")
SRC = r"""
#include "gccd_fp64.h"
#include <cstdio>
int main() {
    double q;
    while (std::fread(&q, sizeof q, 1, stdin) == 1) {
        const double w = gccd::fp64::rsqrt3_pos(q);
        std::fwrite(&w, sizeof w, 1, stdout);
    }
}
"""


def test_rsqrt3_against_40_digits(tmp_path):
    src, exe = tmp_path / "r3.cpp", tmp_path / "r3"
    src.write_text(SRC)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", INC, str(src), "-o",
                    str(exe)], check=True)
    q = 10.0 ** np.random.default_rng(3).uniform(-6.0, 8.0, 4000)
    out = subprocess.run([str(exe)], input=q.tobytes(), capture_output=True, check=True).stdout
    w = np.frombuffer(out, dtype=np.float64)
    assert w.size == q.size
    mp.mp.dps = 40
    ref = [mp.mpf(float(v)) ** (-mp.mpf(3) / 2) for v in q]

    def ulps(x):
        return np.array([float((mp.mpf(float(v)) - r) / mp.mpf(float(np.spacing(float(r)))))
                         for v, r in zip(x, ref)])

    err, ieee = ulps(w), ulps(1.0 / (q * np.sqrt(q)))
    assert np.max(np.abs(err)) <= 1.5
    assert np.sqrt(np.mean(err**2)) <= np.sqrt(np.mean(ieee**2))
