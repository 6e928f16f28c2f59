"""Address arithmetic of the conv patch kernels (csrc/patch_geom.h), compiled
for the host and checked against the memory of the tensors it addresses."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OOB = 0x7FFFFFF0

SRC = """
#include "patch_geom.h"
extern "C" int slot_units(int b) { return xtc::slot_units(b); }
extern "C" int unit_at(int u, int bytes, int start, int oob) {
    return xtc::unit_offset(xtc::unit_entry(u, bytes), start, oob);
}
extern "C" long long store_at(int whole, int pixel, int channel, unsigned first, unsigned row, unsigned oob) {
    const xtc::StoreOffset o = xtc::store_offset(whole, pixel, channel, first, row, oob);
    return (long long)o.lane + o.scalar;
}
extern "C" int no_unit(int start, int oob) { return xtc::unit_offset(-1, start, oob); }
"""


@pytest.fixture(scope="module")
def geom(tmp_path_factory):
    d = tmp_path_factory.mktemp("geom")
    (d / "g.cpp").write_text(SRC)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Werror",
                    "-I" + os.path.join(ROOT, "paper_2512_16512_amd", "csrc"), "-o", str(d / "g.so"),
                    str(d / "g.cpp")], check=True)
    return ctypes.CDLL(str(d / "g.so"))


@pytest.mark.parametrize("N,C,H,W", [(32, 128, 28, 28), (8, 256, 14, 14), (32, 64, 64, 64), (3, 24, 7, 9),
                                     (2, 8, 5, 3), (5, 40, 13, 13), (1, 16, 1, 1)])
@pytest.mark.parametrize("xmis", [0, 2, 8, 14])
def test_input_units_cover_their_run_and_nothing_past_the_tensor(geom, N, C, H, W, xmis):
    """Every unit copied of a run of rows holds bytes of that run, so that none
    lies wholly past the tensor (its last 16-byte unit may be shared with what
    follows), and together they cover it."""
    plane = H * W * 2
    end = xmis + N * C * plane
    for img in (0, N - 1):
        for first, rows in ((0, H), (H - 1, 1), (0, min(3, H)), (H - min(3, H), min(3, H))):
            nb = rows * W * 2
            if nb >= 1 << 15:
                continue
            for ch in (0, 1, C - 1):
                start = xmis + (img * C * H + first) * W * 2 + ch * plane
                got = [geom.unit_at(u, nb, start, OOB) for u in range(geom.slot_units(nb))]
                used = [o for o in got if o != OOB]
                assert used == list(range(start & ~15, start + nb, 16)), (img, first, rows, ch)
                assert max(used) < end and got[len(used):] == [OOB] * (len(got) - len(used))
    assert geom.no_unit(xmis, OOB) == OOB and geom.slot_units(0) == 0


@pytest.mark.parametrize("N,OC,OH,OW", [(1, 16, 100000, 200), (1, 1, 65536, 8000), (1, 3, 21000, 8190),
                                        (1, 27, 99000, 200), (2, 5, 6500, 8100), (3, 70, 28, 28), (1, 64, 8, 8)])
@pytest.mark.parametrize("BM,rows", [(32, [8 * (r >> 2) + (r & 3) for r in range(16)]), (16, range(4))])
def test_stores_outside_the_output_stay_past_it(geom, N, OC, OH, OW, BM, rows):
    """A store of a channel or pixel outside Y goes past the buffer for outputs
    up to the largest accepted one (the offsets of a dropped channel must not
    wrap round into Y), every other one to its element."""
    geom.store_at.argtypes = [ctypes.c_int] * 3 + [ctypes.c_uint] * 3
    geom.store_at.restype = ctypes.c_longlong
    OHW = OH * OW
    span = N * OC * OHW * 4
    assert span <= 0x7FFFFFD0
    for m0 in range(0, OC, BM):
        whole = m0 + BM <= OC
        for lane_oc in range(m0, m0 + BM, 4):
            for row in rows:
                oc = lane_oc + row
                if oc >= m0 + BM:
                    continue
                for img, pix in ((0, 0), (N - 1, OHW - 1), (N, 0)):
                    first = ((img * OC + lane_oc) * OHW + pix) * 4 % 2**32
                    o = geom.store_at(whole, img < N, oc < OC, first, row * OHW * 4 % 2**32, OOB)
                    if img < N and oc < OC:
                        assert o == ((img * OC + oc) * OHW + pix) * 4 < span
                    else:
                        assert OOB <= o < 2**32, (img, pix, oc)
