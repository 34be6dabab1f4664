"""The window of pixels behind the 32-bit offsets of the gathered kernels, against every start of every small grid
(built with the host compiler; needs no GPU)."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

PROGRAM = r"""
#include <cstdio>
#include "grid_window.h"
int main() {
    // grids as they occur: stride 1 and 2 (RH = ceil(H / mul)), one parity of an odd or even side (RH = H / 2 rounded
    // either way, mul = 2), and the gradient's own grid read by the pixels of a parity (mul = 1, RH one less than H)
    long checked = 0;
    for (long H = 1; H <= 7; ++H) for (long W = 1; W <= 5; ++W) for (long mul = 1; mul <= 2; ++mul)
        for (long RH = 1; mul * (RH - 1) < H; ++RH) for (long RW = 1; mul * (RW - 1) < W; ++RW) {
            if (mul * RH + 2 < H || mul * RW + 2 < W) continue;
            const long per = RH * RW;
            for (long rows = 1; rows <= 33; ++rows) {
                long most = 0;
                for (long i = 0; i < per; ++i) {
                    const long e = i + rows - 1;
                    const long first = mul * (i / RW) * W;
                    const long last = ((e / per) * H + mul * (e % per / RW)) * W + mul * (RW - 1);
                    if (last - first + 1 > most) most = last - first + 1;
                }
                ++checked;
                if (abt::grid_window(rows, RH, RW, mul, H, W) != most) {
                    std::printf("rows %ld grid %ld x %ld mul %ld image %ld x %ld: %ld, not %ld\n", rows, RH, RW, mul, H, W,
                                (long)abt::grid_window(rows, RH, RW, mul, H, W), most);
                    return 1;
                }
            }
        }
    // 128 rows of the odd pixels of 3 x 3 images are 128 images: with 2^20 channels no 32-bit offset reaches the last
    if (abt::grid_window(128, 1, 1, 2, 3, 3) * (1l << 20) * 2 < 0x7ffffff0l) return 2;
    if (abt::grid_window(64, 0, 3, 1, 4, 4) != 0) return 3;
    std::printf("%ld\n", checked);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_window_is_the_largest_over_all_starts(tmp_path):
    src = tmp_path / "window.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "window")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2405_01067_amd", "csrc"), str(src), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 1000


FITS = r"""
#include <cstdio>
#include "grid_window.h"
int main() {
    int accepted = 0;
    for (int R = 32; R <= 192; R += 32)
        for (long pixels = 1; pixels <= 300; ++pixels) {
            const long slots = (pixels + 7) / 8 * 8, bytes = 2l * R * 64 * 2 + (slots + 1) * 64 * 2;
            if (abt::window_fits(R, pixels) != (pixels <= 256 && bytes <= 80 * 1024)) { std::printf("R %d, %ld pixels\n", R, pixels); return 1; }
            accepted += abt::window_fits(R, pixels);
        }
    std::printf("%d\n", accepted);
    return abt::window_fits(192, 248) && !abt::window_fits(192, 249) && abt::window_fits(160, 256) ? 0 : 2;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_windows_leave_room_for_two_work_groups(tmp_path):
    src = tmp_path / "fits.cpp"
    src.write_text(FITS)
    exe = str(tmp_path / "fits")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2405_01067_amd", "csrc"), str(src), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) == 5 * 256 + 248
