"""The library's own host code on the CPU: fake_hip.c stands in for the HIP
runtime (no GPU, allocations that can be made to fail, recorded launches), so
that buffer handling after a failed allocation and the grids of very large
lattices are checked without running a kernel."""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_1907_00641_amd", "libpam_lattice.so")

pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc not available")

# run in a process of its own, which loads the stand-in first and no torch
DRIVER = """
import ctypes, json, re, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
shim.fake_log.restype = ctypes.c_char_p
shim.fake_fail_above.argtypes = [ctypes.c_uint64]
vp, i64, i32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32
L.pam_lattice_build.argtypes = [vp, i64, i32, vp, ctypes.POINTER(vp)]
L.pam_lattice_set_capacity.argtypes = [vp, i64, i32]
L.pam_filter_fwd.argtypes = [vp, vp, i32, ctypes.c_uint32, vp, vp]
FEAT = vp(0x200000)
h = vp(None)

def build(n, d, vertices, buckets=200):
    "(status, [(kernel, grid x, block x, refused)])"
    shim.fake_clear()
    shim.fake_outcome(vertices, 0, buckets)
    st = L.pam_lattice_build(FEAT, n, d, None, ctypes.byref(h))
    rows = []
    for line in shim.fake_log().decode().splitlines():
        if line.startswith("malloc"):
            continue
        name, gx, gy, gz, bx = line.split()[:5]
        rows.append((re.search("(k_[a-z0-9_]+?)(ILi|E|$)", name).group(1), int(gx), int(bx), line.endswith("refused")))
    return st, rows

def mallocs():
    return [int(line.split()[1]) for line in shim.fake_log().decode().splitlines() if line.startswith("malloc")]

out = {}
exec(sys.argv[3])
print(json.dumps(out))
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not os.path.exists(LIB):
        from paper_1907_00641_amd.build import build_library

        build_library()
    shim = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.c"), "-o", shim, "-ldl"], check=True)

    def go(body):
        r = subprocess.run([sys.executable, "-c", DRIVER, shim, LIB, body], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
        return json.loads(r.stdout.splitlines()[-1])

    return go


def test_build_launches(run):
    """First build, then a rebuild, which needs no range pass."""
    out = run("out['first'] = build(4000, 3, 100)\nout['again'] = build(4000, 3, 100)")
    chain = ["k_insert", "k_starts", "k_scatter", "k_sorted_tiles", "k_compact", "k_resolve"]
    assert out["first"][0] == 0 and out["again"][0] == 0
    assert [r[0] for r in out["first"][1]][:8] == ["k_range", "k_layout"] + chain
    assert [r[0] for r in out["again"][1]] == chain


def test_neighbour_items_of_large_lattices(run, tmp_path):
    """340 million vertices at d = 12: 4.4e9 neighbour items, more than 32
    bits index and more work items than one launch may have."""
    out = run("out['r'] = [build(30000000, 12, 340000000), build(30000000, 12, 340000000)]")
    for st, rows in out["r"]:
        assert st == 0 and not any(r[3] for r in rows), rows
    # every item exactly once, for small extents by enumeration and for the
    # large one at its ends
    src = tmp_path / "items.cpp"
    src.write_text(r'''
#include "pam_grid.h"
#include <cstdio>
#include <vector>
using namespace pam;
static int fail(const char *what, long long a, long long b) { printf("%s %lld %lld\n", what, a, b); return 1; }
int main()
{
    for (int dirs : {2, 6, 17})
        for (int64_t M : {1, 255, 256, 257, 5000})
            for (int64_t estimate : {(int64_t)1, M, 4 * M}) {
                const unsigned per = nbr_blocks_per_dir(estimate), blocks = per * (unsigned)dirs;
                std::vector<int> seen(M * dirs, 0);
                for (unsigned b = 0; b < blocks; ++b)
                    for (int t = 0; t < kGridBlock; ++t)
                        for (int64_t m = nbr_first(b, per, t); m < M; m += nbr_stride(per)) {
                            const int64_t at = nbr_entry(nbr_dir(b, per), m, M);
                            if (at < 0 || at >= M * dirs) return fail("outside", at, M);
                            ++seen[at];
                        }
                for (int64_t e = 0; e < M * dirs; ++e)
                    if (seen[e] != 1) return fail("entry", e, seen[e]);
            }
    const int64_t M = 340000000;
    const int dirs = 13;
    const unsigned per = nbr_blocks_per_dir(M), blocks = per * dirs;
    if ((int64_t)blocks * kGridBlock >= (int64_t)1 << 32) return fail("grid", blocks, 0);
    int64_t last = -1, m = nbr_first(blocks - 1, per, kGridBlock - 1);
    if (nbr_dir(blocks - 1, per) != dirs - 1) return fail("direction", nbr_dir(blocks - 1, per), 0);
    for (; m < M; m += nbr_stride(per)) last = nbr_entry(dirs - 1, m, M);
    if (last <= ((int64_t)1 << 32) || last >= M * dirs) return fail("last entry", last, M * dirs);
    return 0;
}
''')
    exe = tmp_path / "items"
    csrc = os.path.join(os.path.dirname(LIB), "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", csrc, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_tile_hash_holds_every_row(tmp_path):
    """A tile's LDS hash has room for as many rows as contributions, with
    probes of bounded length: tiles of points that share no bucket, whose
    vertices step down the coordinates in random orders."""
    src = tmp_path / "hash.cpp"
    src.write_text(r'''
#include "pam_grid.h"
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>
using namespace pam;
int main()
{
    std::mt19937 rng(5);
    for (int d = 1; d <= 16; ++d) {
        const int T = tile_points(d), H = tile_slots(d);
        long probes = 0, longest = 0, keys = 0;
        for (int rep = 0; rep < 8; ++rep) {
            std::vector<uint32_t> slot(H, ~0u);
            std::vector<int> order(d + 1);
            for (int p = 0; p < T; ++p) {
                for (int c = 0; c <= d; ++c) order[c] = c;
                std::shuffle(order.begin(), order.end(), rng);
                uint32_t key = (uint32_t)p << (d + 1);
                for (int k = 0; k <= d; ++k) {
                    if (k) key |= 1u << order[k];
                    uint32_t h = tile_hash(key, H);
                    long n = 1;
                    for (; slot[h] != ~0u; h = h + 1 < (uint32_t)H ? h + 1 : 0)
                        if (++n > H) { printf("d=%d: no room for row %ld\n", d, keys); return 1; }
                    slot[h] = key;
                    probes += n, ++keys, longest = std::max(longest, n);
                }
            }
        }
        printf("d=%d mean %.1f longest %ld\n", d, (double)probes / keys, longest);
        if ((double)probes / keys > 12 || longest > H / 2) return 2;
    }
    return 0;
}
''')
    exe = tmp_path / "hash"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(os.path.dirname(LIB), "csrc"), str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_range_pass_after_a_failed_allocation(run):
    """A build whose vertex table grows moves the bucket table too; when it
    then runs out of memory for the points, the next build finds a bucket
    table that nothing has emptied, and must not take it as empty."""
    out = run("""
out['grow'] = [build(4000, 3, 100), build(4000, 3, 200000)]
shim.fake_fail_above(1 << 25)
out['fails'] = build(1000000, 3, 200000)
shim.fake_fail_above((1 << 64) - 1)
out['next'] = build(4000, 3, 100)
out['again'] = build(4000, 3, 100)
""")
    assert [st for st, _ in out["grow"]] == [0, 0]
    st, rows = out["fails"]
    assert st == 2 and rows == []  # out of memory, before any launch
    st, rows = out["next"]
    assert st == 0 and [r[0] for r in rows][:3] == ["k_range", "k_layout", "k_insert"]
    st, rows = out["again"]
    assert st == 0


def test_largest_table_capacity(run):
    """pam_lattice_set_capacity takes up to 2^34 slots; no launch of the
    build may then exceed what a launch may have."""
    out = run("""
build(4000, 3, 100)
out['set'] = L.pam_lattice_set_capacity(h, 1 << 34, 1)
out['large'] = build(4000, 3, 100)
""")
    st, rows = out["large"]
    assert out["set"] == 0
    assert st == 0 and not any(r[3] for r in rows), rows


def test_shared_allocation_of_large_buffers_only(run):
    """The four lattice buffers of a forward call: allocations below 2 MB
    cost the host about 1 us each and stay apart, from 2 MB on (tens to
    hundreds of us each) they share one."""
    out = run("""
for name, vertices in (('small', 16000), ('large', 17000)):
    h = vp(None)
    build(100000, 3, vertices)
    shim.fake_clear()
    out[name] = [L.pam_filter_fwd(h, vp(0x40000000), 32, 0, vp(0x60000000), None), mallocs()]
""")
    assert out["small"] == [0, [16000 * 128] * 4]
    st, sizes = out["large"]
    assert st == 0 and len(sizes) == 1 and sizes[0] >= 4 * 17000 * 128


def test_second_build_needs_no_range_pass(run):
    """A new handle guesses its bucket table from the point count.  A guess
    of at most 2^16 slots is kept however few buckets there are, so that the
    second build finds it emptied; a larger one that is far too large shrinks
    once, and the build after that is fast."""
    out = run("""
for name, n in (('small', 32768), ('mid', 262144), ('large', 2000000)):
    h = vp(None)
    out[name] = [[r[0] for r in build(n, 3, 900, 300)[1]] for _ in range(3)]
h = vp(None)
out['wide'] = [[r[0] for r in build(32768, 3, 900, 20000)[1]] for _ in range(3)]  # over half full
""")
    takes_range = {k: ["k_range" in rows for rows in v] for k, v in out.items()}
    assert takes_range == {"small": [True, False, False], "mid": [True, False, False], "large": [True, True, False],
                           "wide": [True, True, False]}
