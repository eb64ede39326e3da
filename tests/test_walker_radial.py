"""Walks along lines through the grid's centre, built for the host: the square of
their distance from it is rounding noise of either sign, and the walk has to stay in
its rows and columns all the same."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2110_15640_amd", "csrc")
ROCM = "/opt/rocm/include"

SOURCE = r"""
#define __builtin_amdgcn_rcp(x) (1.0 / (x))
#define __builtin_amdgcn_rsq(x) (1.0 / sqrt(x))
#include "device_common.hpp"
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
using namespace mcrt;
using namespace mcrt::dev;
static long bad = 0, walks = 0;
template <bool FAST, bool RAYS>
void radial(int nlon, int nlat, int nlay, int n, double tilt)
{
    std::vector<double> r, lat, lon, c2;
    std::vector<double2> f;
    for (int k = 0; k <= nlay; ++k) r.push_back(7e9 + 7e8 * k / nlay);
    for (int e = 0; e <= nlat; ++e) lat.push_back(-0.5 * M_PI + M_PI * e / nlat), c2.push_back(cos(lat[e]) * cos(lat[e]));
    for (int e = 0; e <= nlon; ++e) lon.push_back(-M_PI + 2.0 * M_PI * e / nlon);
    GridDev g{};
    g.nlon = nlon; g.nlat = nlat; g.nlay = nlay;
    g.lat_base = nlay; g.lon_base = nlay + nlat; g.lat_c2 = c2.data();
    for (int k = 0; k < nlay; ++k) f.push_back({r[k], r[k + 1]});
    for (int j = 0; j < nlat; ++j) f.push_back({j ? sin(lat[j]) : -2.0, j + 1 < nlat ? sin(lat[j + 1]) : 2.0});
    for (int e = 0; e <= nlon; ++e) f.push_back({sin(lon[e % nlon]), cos(lon[e % nlon])});
    g.faces = f.data();
    std::mt19937_64 rng(5);
    std::uniform_real_distribution<double> U(0.0, 1.0);
    for (int q = 0; q < n; ++q, ++walks) {
        const int i = rng() % nlon, j = rng() % nlat, k = rng() % nlay;
        const double rr = r[k] + U(rng) * (r[k + 1] - r[k]);
        // clear of the cell's faces by a part in 1e3 of it, which a line this close to radial does not leave
        const double s0 = sin(lat[j]), sl = s0 + (0.001 + 0.998 * U(rng)) * (sin(lat[j + 1]) - s0), cl = sqrt(1.0 - sl * sl);
        const double lo = lon[i] + (0.001 + 0.998 * U(rng)) * (lon[i + 1] - lon[i]);
        const double px = rr * cl * cos(lo), py = rr * cl * sin(lo), pz = rr * sl;
        const double sgn = q & 1 ? 1.0 : -1.0;  // outward to the top, inward to the planet
        double dx = sgn * px / rr + tilt * (U(rng) - 0.5), dy = sgn * py / rr + tilt * (U(rng) - 0.5),
               dz = sgn * pz / rr + tilt * (U(rng) - 0.5);
        const double norm = sqrt(dx * dx + dy * dy + dz * dz);
        dx /= norm; dy /= norm; dz /= norm;
        Walker w;
        wk_start<FAST, GEO_SPHERE>(g, w, px, py, pz, dx, dy, dz, i, j, k);
        bool out = false, wrong = false;
        int m = 0;
        for (; m < 4 * nlay + 8 && !out && !wrong; ++m) {
            const CrossKind x = wk_next<GEO_SPHERE>(w);
            Walker next = w;  // the row and column that the crossing would read
            next.j += x.cone ? next.dj : 0;
            if (!(x.t < 1e11) || next.j < 0 || next.j >= nlat) { wrong = true; break; }
            const CrossIn in = wk_cross_begin<GEO_SPHERE>(g, w, x);
            out = !in.inside;
            wrong = w.j != j || w.i != i;
            if (!out) wk_cross_end<FAST, GEO_SPHERE, RAYS>(g, w, x, in, RAYS);
        }
        bad += wrong || !out || (w.k < 0) != (sgn < 0.0);
    }
}
int main(int, char** a)
{
    const int nlon = atoi(a[1]), nlat = atoi(a[2]), nlay = atoi(a[3]);
    const double tilt = atof(a[4]);
    radial<false, false>(nlon, nlat, nlay, 20000, tilt);
    radial<true, false>(nlon, nlat, nlay, 20000, tilt);
    radial<false, true>(nlon, nlat, nlay, 20000, tilt);
    radial<true, true>(nlon, nlat, nlay, 20000, tilt);
    printf("%ld wrong of %ld\n", bad, walks);
    return bad != 0;
}
"""


@pytest.fixture(scope="module")
def walker(tmp_path_factory):
    if not shutil.which("g++") or not os.path.exists(os.path.join(ROCM, "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP headers")
    d = tmp_path_factory.mktemp("radial")
    (d / "w.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-w", "-O2", "-std=gnu++17", "-ffp-contract=off", "-mfma", "-D__HIP_PLATFORM_AMD__",
                           "-D__umulhi(a,b)=((uint32_t)(((uint64_t)(a)*(uint64_t)(b))>>32))", "-I" + ROCM, "-I" + CSRC,
                           str(d / "w.cpp"), "-o", str(d / "w")])
    return str(d / "w")


# tilt: up to a direction's rounding, and around the distance at which its square is noise (1e-8)
@pytest.mark.parametrize("tilt", ["0", "1e-16", "1e-12", "1e-9", "1e-8", "1e-7"])
@pytest.mark.parametrize("shape", [(1, 1, 12), (3, 2, 5), (45, 23, 7), (128, 64, 20), (8, 2, 50)])
def test_radial_walks_keep_their_column(walker, shape, tilt):
    p = subprocess.run([walker] + [str(v) for v in shape] + [tilt], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout + p.stderr
