"""The grid walk of the ray cast, compiled for the host: its face crossings
against 64 bits, from inside the grid and from far outside, on every axis
length a grid may have."""
import os
import subprocess

import numpy as np
import pytest

from paper_2312_11841_amd import build

# Reads rays (o, d) and a grid per ray from a file of floats, enters the walk
# and prints, per ray and moving axis, the crossing distance of a face: the
# ray's own t as the walk has it, and the face's index.
PROGRAM = r"""
#include <stdio.h>
#include <vector>
#include "mixrt_mesh.hpp"
int main(int argc, char **argv)
{
    FILE *in = fopen(argv[1], "rb"), *out = fopen(argv[2], "wb");
    float v[16];
    while (fread(v, sizeof(float), 16, in) == 16) {
        mixrt::MeshGridK g{};
        for (int a = 0; a < 3; ++a) {
            g.lo[a] = v[6 + a];
            g.hi[a] = v[9 + a];
            g.n[a] = (int)v[12 + a];
            const double cell = ((double)g.hi[a] - (double)g.lo[a]) / g.n[a];
            g.cell[a] = (float)cell;
            g.inv_cell[a] = (float)(1.0 / cell);
        }
        mixrt::Walk w;
        float t_in, r[8] = {0};
        r[0] = mixrt::walk_enter(g, v, v + 3, w, t_in);
        if (r[0]) {
            r[1] = t_in;
            // to a cell of the walk's choice: a fraction v[15] of the axis
            for (int a = 0; a < 3; ++a)
                w.c[a] = floorf(v[15] * (float)(g.n[a] - 1) + 0.5f);
            mixrt::walk_faces(w);
            for (int a = 0; a < 3; ++a) {
                r[2 + a] = w.tn[a];
                r[5 + a] = w.c[a] + (w.st[a] > 0.0f ? 1.0f : 0.0f);
            }
        }
        fwrite(r, sizeof(float), 8, out);
    }
    fclose(out);
    return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("walk")
    src, exe = d / "walk.cpp", d / "walk"
    src.write_text(PROGRAM)
    flags = [f for f in build.FLAGS if f != "-fPIC" and not f.startswith("--offload")]
    i = flags.index("-mllvm")                       # (an option of the device compiler)
    del flags[i:i + 2]
    r = subprocess.run([build.HIPCC, "--offload-host-only", *flags, "-I", build.INCLUDE, "-I",
                        build.CSRC, "-x", "hip", str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(rows):
        np.ascontiguousarray(rows, np.float32).tofile(d / "in")
        subprocess.run([str(exe), str(d / "in"), str(d / "out")], check=True)
        return np.fromfile(d / "out", np.float32).reshape(len(rows), 8).astype(np.float64)

    return run


@pytest.mark.parametrize("distance", [0.0, 1.0, 10.0, 100.0, 1e4])
@pytest.mark.parametrize("n", [1, 64, 256, 1024])
@pytest.mark.parametrize("place", [0.0, 0.9])
def test_face_crossings_stay_within_the_pad(walk, distance, n, place):
    """Where the ray o + t d, followed exactly, is when the walk says that it
    crosses a face, in cells of that axis.  A crossing is a product and a
    quotient of numbers up to n cells, a dozen roundings in all of 2^-24 each
    (the entry point's two and the scaling's three, the face's sum, the
    reciprocal's and the product's), most at half that: n 2^-21.  Triangles
    are listed in cells padded by 1/500, which 1024 cells keep four times
    over.  The box lies at the origin, and off it by nine tenths of its size
    (its own coordinates then round alike).  From outside, t_in itself is
    exact as a number: t is t_in plus the walk's distance."""
    rng = np.random.default_rng(int(distance) + n)
    rows = np.zeros((4000, 16), np.float32)
    m = len(rows)
    lo = (place + rng.uniform(-0.05, 0.05, (m, 3))).astype(np.float32)
    hi = (lo + rng.uniform(0.5, 1.0, (m, 3))).astype(np.float32)
    # from a point at that many extents through one inside the box
    inside = lo + (hi - lo) * rng.uniform(0.02, 0.98, (m, 3))
    d = rng.normal(size=(m, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    rows[:, 0:3] = inside - distance * d
    rows[:, 3:6] = d
    rows[:, 6:9], rows[:, 9:12] = lo, hi
    rows[:, 12:15] = n
    rows[:, 15] = rng.uniform(0, 1, m)
    r = walk(rows)
    e = rows.astype(np.float64)
    met = r[:, 0] > 0
    assert met.mean() > (0.999 if distance < 1e3 else 0.99)
    cell = (e[:, 9:12] - e[:, 6:9]) / n
    t = r[:, 1:2] + r[:, 2:5]
    at = (e[:, 0:3] + t * e[:, 3:6] - e[:, 6:9]) / cell
    # only faces the ray meets near the box: elsewhere t outgrows the grid
    near = met[:, None] & (np.abs(r[:, 2:5]) < 3.0)
    err = np.abs(at - r[:, 5:8])[near].max()
    print(f"n {n} distance {distance:g} place {place}: {err:.2e} of a cell")
    assert err <= n * 2.0 ** -21
