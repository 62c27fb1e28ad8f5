"""Which planes along z the kernels' blocks read: csrc/pp_planes.h is plain C++,
compiled here for the host and taken through every case of small grids."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2012_11744_amd", "csrc")


def run_host(tmp_path, body):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include <initializer_list>\n#include "pp_planes.h"\nusing namespace pp;\n' + body)
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)])
    return subprocess.run([str(exe)], capture_output=True, text=True)


def test_two_sweep_march_stays_inside_the_array(tmp_path):
    """Every plane that a march loads, for every storage type, nz from the least
    (8) on, chunk length, wall and loop form, is inside the array or not read, and
    every plane that the chunk's output needs is the right one."""
    r = run_host(tmp_path, r'''
int main()
{
    int far = 0;
    for (int word : {2, 4, 8})
        for (int nz = 8; nz <= 40; ++nz)
            for (int kz = 2; kz <= nz; ++kz)
                for (int k0 = 0; k0 < nz; k0 += kz)
                    for (int wall = 0; wall < 2; ++wall)
                        for (int whole = 0; whole < 2; ++whole) {
                            const int k1 = k0 + kz < nz ? k0 + kz : nz, last = two_sweep_last_plane(k1);
                            const int fpd = two_sweep_depth(word), fnb = two_sweep_unroll(word);
                            int k = two_sweep_first(k0), end = k;
                            while (end <= two_sweep_end(k1))
                                end += whole ? fnb : 1;
                            // the prologue loads from k0 - 4, step k plane k + 1 + fpd
                            for (int q = k0 - 4; q <= end - 1 + 1 + fpd; ++q) {
                                int qw = -1;
                                const bool there = march_plane<true>(q, nz, wall, last, qw);
                                if (there && (qw < 0 || qw >= nz)) {
                                    std::printf("word %d nz %d kz %d k0 %d: plane %d read as %d\n",
                                                word, nz, kz, k0, q, qw);
                                    return 1;
                                }
                                const bool out = q < 0 || q >= nz;
                                if (q <= k1 + 3 && (there != !(wall && out) ||
                                                    (there && qw != (q + nz) % nz))) {
                                    std::printf("nz %d kz %d k0 %d: plane %d is wrong\n", nz, kz, k0, q);
                                    return 1;
                                }
                                // one resource for the whole array (at most 2^31 - 16 bytes):
                                // offsets past its end do not wrap around 32 bits
                                march_plane<false>(q, nz, wall, last, qw);
                                if (qw < 0 || (qw + 1.0) * (0x7ffffff0u / nz) > 4294967295.0) {
                                    std::printf("word %d nz %d kz %d k0 %d: offset of %d wraps\n",
                                                word, nz, kz, k0, q);
                                    return 1;
                                }
                                far = q - nz > far ? q - nz : far;
                            }
                            if (k != k0 - 3 || end <= k1 + 2)
                                return 2;
                        }
    return far >= 10 ? 0 : 3;   // the case of nz = 8: ten planes past the end
}
''')
    assert r.returncode == 0, r.stdout


def test_planes_per_block(tmp_path):
    """The blocks along z cover the grid, none of them empty, and where the order of
    the sums is fixed they hold 8 planes whatever nz is (the last what is left)."""
    r = run_host(tmp_path, r'''
int main()
{
    for (int nz = 1; nz <= 600; ++nz)
        for (int most = 1; most <= 8; most *= 2)
            for (std::size_t xy : {1, 7, 64, 300, 5000}) {
                const int kz = walk_planes(nz, xy, most), gz = (nz + kz - 1) / kz;
                const int pl = planes_of(nz, gz, false);
                if (kz < 1 || kz > most || pl > kz || gz * pl < nz || (gz - 1) * pl >= nz)
                    return 1;
                const int g8 = (nz + FIXED_PLANES - 1) / FIXED_PLANES;
                if (FIXED_PLANES != 8 || planes_of(nz, g8, true) != 8)
                    return 2;
            }
    return 0;
}
''')
    assert r.returncode == 0
