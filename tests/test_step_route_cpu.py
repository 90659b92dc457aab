"""The rules of csrc/step_route.h, compiled for the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, body):
    src, exe = tmp_path / "route.cpp", tmp_path / "route"
    src.write_text('#include "step_route.h"\n#include <stdio.h>\n#include <vector>\nusing namespace pcpic;\n'
                   "#define CHECK(x) do { if (!(x)) { printf(\"line %d: %s\\n\", __LINE__, #x); return 1; } } while (0)\n"
                   "int main()\n{\n" + body + "\n    return 0;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_1011_6330_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


needs_gxx = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@needs_gxx
def test_push_order_takes_each_tile_once_on_its_xcd(tmp_path):
    """Both orders cover every tile exactly once within the launched blocks, whatever the
    capacity's grid; a tile stays on the XCD (block index mod 8) of the ascending order; and
    the descending one starts within 8 tiles of the last."""
    _run(tmp_path, """
    for (int64_t tiles = 0; tiles < 70; ++tiles)
        for (int64_t cap = tiles; cap < tiles + 20; ++cap)
            for (int rev = 0; rev < 2; ++rev) {
                std::vector<int> seen((size_t)tiles, 0);
                for (int64_t k = 0; k < (int64_t)push_blocks(cap); ++k) {
                    const int64_t t = push_tile(k, tiles, rev);
                    if (t < 0 || t >= tiles) continue;
                    ++seen[(size_t)t];
                    CHECK(t % XCDS == k % XCDS);
                    if (rev && k < XCDS) CHECK(t >= tiles - XCDS);
                }
                for (int s : seen) CHECK(s == 1);
            }
""")


@needs_gxx
def test_push_access_rule(tmp_path):
    _run(tmp_path, """
    CHECK(push_nontemporal(0) && push_nontemporal((int64_t)32 << 20) && !push_nontemporal(((int64_t)32 << 20) + 1));
    CHECK(!push_nontemporal((int64_t)1 << 30) && push_nontemporal(((int64_t)1 << 30) + 1));
    CHECK(push_nontemporal(((int64_t)1 << 62)));
""")


@needs_gxx
def test_expected_slots(tmp_path):
    """The density's, the capacity's or the slots last seen, whichever decides."""
    _run(tmp_path, """
    CHECK(expected_slots(20.0, 20000, 14000000, 0) == 800000);
    CHECK(expected_slots(20.0, 20000, 500000, 0) == 500000);
    CHECK(expected_slots(20.0, 20000, 14000000, 12000000) == 12000000);
    CHECK(expected_slots(20.0, 20000, 14000000, 700000) == 800000);
    CHECK(expected_slots(1e300, 20000, 4096, 0) == 4096);
    CHECK(expected_slots(20.0, 20000, 14000000, 12000000) > fuse_slots(true, false));
    CHECK(fuse_slots(false, false) < fuse_slots(false, true) && fuse_slots(false, true) < fuse_slots(true, true));
""")


@needs_gxx
def test_scatter_blocks(tmp_path):
    """The tiles' blocks, unless the key counts need more to be cleared 2048 to a block."""
    _run(tmp_path, """
    CHECK(scatter_blocks(4, 2048) == 4 && scatter_blocks(4, 4 * 2048) == 4 && scatter_blocks(4, 4 * 2048 + 1) == 5);
    CHECK(scatter_blocks(1, 1 << 20) == 512 && scatter_blocks(40000, 1 << 20) == 40000);
""")


@needs_gxx
def test_jump_rules(tmp_path):
    """Slots in order have jumps only where a wave spans more than 63 cells; the limits fall
    with the cells, and where most of the slots jump."""
    _run(tmp_path, """
    CHECK(ordered_jumps(0, 1000, false) == 0 && ordered_jumps(1000000, 65536, false) == 0);
    CHECK(ordered_jumps(300000, 100000, true) > 0 && ordered_jumps(300000, 100000, false) == 0);
    CHECK(ordered_jumps(20000, 65536, false) > 6000 && ordered_jumps(20000, 65536, false) < 8000);
    CHECK(ordered_jumps(10, 1 << 20, false) <= 10);
    CHECK(jump_stride(1) == 1 && jump_stride(256 * 1024) == 1 && jump_stride(256 * 1024 + 1) == 2);
    for (int f32 = 0; f32 < 2; ++f32) {
        int64_t last = INT64_MAX;
        for (int64_t n : {700, 4095, 4096, 32767, 32768, 131071, 131072, 1 << 24}) {
            const int64_t few = most_jumps(1000, 1000000, n, f32), most = most_jumps(1000000, 1000000, n, f32);
            CHECK(most <= few && few <= last && most > 0);
            last = few;
        }
    }
    CHECK(400000 > most_jumps(400000, 400000, 65536, false));      // 35.3 us a step in separate kernels, 41.8 fused
    CHECK(98000 <= most_jumps(98000, 100000, 10000, false));       // 15.0 / 13.8
    CHECK(7000 <= most_jumps(7000, 20000, 65536, false));          // 8.1 / 6.9
    CHECK(19800 > most_jumps(19800, 20000, 65536, true));          // 9.9 / 12.4
""")
