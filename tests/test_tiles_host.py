"""The tile table of the time-blocked kernels (host code, compiled here): every
tile's node list starts where the one before ends, also where the lists of a
batch hold more than 2^31 entries."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "lbm_tiles.hpp"
struct I { int nx, ny; };
// args: ms big nx ny n xper yper
int main(int c, char **v) {
    if (c != 8) return 2;
    lbm::Blocks B;
    B.ms = atoi(v[1]);
    B.big = atoi(v[2]);
    const bool xper = atoi(v[6]), yper = atoi(v[7]);
    std::vector<I> inst(atoi(v[5]), I{atoi(v[3]), atoi(v[4])});
    for (const I &i : inst) B.count(i.nx, i.ny, xper, yper);
    const std::vector<lbm::MTileDesc> t = lbm::tile_table(B, inst, xper, yper);
    if ((int)t.size() != B.n_tiles) return 3;
    long long at = 0;
    for (const lbm::MTileDesc &e : t) {
        // the region, clipped at the edges of an axis that is not periodic
        long long n[2];
        const int at0[2] = {e.x0, e.y0}, size[2] = {inst[e.b].nx, inst[e.b].ny}, tile[2] = {B.tx(), B.ty()};
        for (int a = 0; a < 2; ++a) {
            n[a] = 0;
            const int last = at0[a] + tile[a] < size[a] ? at0[a] + tile[a] : size[a];
            for (int p = at0[a] - B.ms; p < last + B.ms; ++p) n[a] += (a ? yper : xper) || (p >= 0 && p < size[a]);
        }
        if (e.list != at || n[0] > B.ex() || n[1] > B.ey()) return 4;
        at += n[0] * n[1];
    }
    if (at != B.n_entries) return 5;
    printf("%lld\n", at);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("tiles")
    (d / "t.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2310_00810_amd", "csrc"),
                    str(d / "t.cpp"), "-o", str(d / "t")], check=True)
    return str(d / "t")


@pytest.mark.parametrize("ms,big,nx,ny,n,xper,yper", [
    (6, 0, 9, 5, 3, 0, 0), (6, 0, 20, 4, 1, 1, 1), (5, 0, 233, 160, 2, 0, 1), (4, 0, 401, 301, 1, 1, 0),
    (5, 1, 655, 317, 2, 0, 0), (5, 1, 1024, 1024, 1300, 0, 1)])
def test_lists_are_adjacent(program, ms, big, nx, ny, n, xper, yper):
    r = subprocess.run([program] + [str(v) for v in (ms, big, nx, ny, n, xper, yper)], capture_output=True, text=True)
    assert r.returncode == 0, r.returncode
    if n >= 1300:
        assert int(r.stdout) > 2 ** 31
