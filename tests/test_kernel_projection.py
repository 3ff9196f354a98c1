"""The two segment searches of the raceline projection (sgtp.hip: `project`, rows read in batches,
and `project_ahead`, the first rows read before the state is known), built for the CPU from the
kernel source and compared with the walk they stand for, one row at a time: forwards while the
next row lies behind the point, backwards while the segment's own row lies ahead of it, at most
max_moves moves inside the window.  A walk that moved forwards never turns back, also where the
rows' normals cross (a point beyond the inside of a tight corner)."""

import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_25388_amd", "csrc",
                   "sgtp.hip")
NPF = 6  # rows read ahead by the kernels

SHIM = r"""
#include <cmath>
#include <type_traits>
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_sqrtf sqrtf
#define __builtin_amdgcn_rsqf(x) (1.0f / sqrtf(x))
struct float4 { float x, y, z, w; };
static int min(int a, int b) { return a < b ? a : b; }
static int max(int a, int b) { return a > b ? a : b; }
static float fast_rcp(float x) { return 1.0f / x; }
"""

ENTRY = r"""
// which 0: the plain walk, 1: project, 2: project_ahead; out: segment, limit per point
extern "C" void search(const float4 *nodes, int W, int max_moves, int n, const float *xy, const int *seg0, int which,
                       int *seg, int *limit) {
    for (int i = 0; i < n; ++i) {
        const float X = xy[2 * i], Y = xy[2 * i + 1];
        int s = seg0[i];
        if (which == 0) {
            auto g = [&](int k) { return ahead_of(nodes[2 * k], X, Y); };
            int moves = 0;
            while (moves < max_moves && s + 1 <= W - 2 && g(s + 1) > 0.0f) { ++s; ++moves; }
            if (s == seg0[i]) while (moves < max_moves && s > 0 && g(s) < 0.0f) { --s; ++moves; }
            seg[i] = s;
            limit[i] = !(g(s) >= 0.0f && g(s + 1) <= 0.0f);
        } else {
            const Foot f = which == 1 ? project(nodes, W, max_moves, X, Y, 32 * s)
                                      : project_ahead<NPF>(nodes, W, max_moves, X, Y, s, read_ahead<NPF>(nodes, W, s));
            seg[i] = which == 1 ? f.seg / 32 : f.seg;
            limit[i] = f.limit;
        }
    }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    text = open(SRC).read()
    a = text.index("__device__ __forceinline__ float ahead_of(")
    b = text.index("// ------", text.index("Foot project_ahead("))
    d = tmp_path_factory.mktemp("projection")
    (d / "p.cpp").write_text(SHIM + text[a:b] + ENTRY.replace("NPF", str(NPF)))
    subprocess.check_call([shutil.which("g++") or "g++", "-O1", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared",
                           "-Wno-unknown-pragmas", "-o", str(d / "p.so"), str(d / "p.cpp")])
    return C.CDLL(str(d / "p.so"))


def _search(lib, rows, W, max_moves, xy, seg0, which):
    n = len(seg0)
    # three rows past the window: `project` reads them in a batch and does not use them
    buf = np.zeros((W + 4, 8), np.float32)
    buf[:W, :4] = rows
    buf[:, 4:6] = 5.0
    xy, seg0 = np.ascontiguousarray(xy, np.float32), np.ascontiguousarray(seg0, np.int32)
    seg, lim = np.zeros(n, np.int32), np.zeros(n, np.int32)
    p = lambda v: v.ctypes.data_as(C.c_void_p)
    lib.search(p(buf), W, max_moves, n, p(xy), p(seg0), which, p(seg), p(lim))
    return seg, lim


def _rows_of_signs(signs):
    """Rows whose distance ahead of the origin has the given signs (normal (0, 1): minus x)."""
    return np.array([[-s, 0.0, 0.0, 1.0] for s in signs], np.float32)


@pytest.mark.parametrize("signs,start,max_moves,want", [
    ([-1] + [1] * 5 + [-1] * 4, 0, 64, 5),           # a whole batch passed, the next row not
    ([-1] * 3 + [1] * 5 + [-1] * 4, 2, 64, 7),       # the same with segments behind
    ([-1] * 3 + [1] * 10 + [-1] * 4, 2, 64, 12),     # two batches
    ([-1] * 3 + [1] * 5 + [-1] * 4, 2, 5, 7),        # the budget used up at the batch's end
    ([-1] * 3 + [1] * 4 + [-1] * 4, 2, 3, 5),
    ([1, 1, -1, -1, 1], 3, 64, 1),                   # no room forwards (the window's last segment): backwards
    ([1, 1, -1, -1, 1], 3, 1, 2),
    ([1, 1, -1, -1, -1, -1], 3, 64, 1),
    ([1, 1, 1, 1, 1, 1, 1, 1, 1], 0, 64, 7),
])
def test_rows_of_given_signs(lib, signs, start, max_moves, want):
    rows = _rows_of_signs(signs)
    got = [int(_search(lib, rows, len(signs), max_moves, [[0.0, 0.0]], [start], w)[0][0]) for w in range(3)]
    assert got == [want] * 3


def _rounded_rectangle(radius, ds, a=20.0, b=12.0):
    """Rows (x, y, nx, ny) along a rectangle with rounded corners, anticlockwise."""
    pts = []
    for k, (cx, cy) in enumerate([(a, -b), (a, b), (-a, b), (-a, -b)]):
        cx, cy = cx - np.sign(cx) * radius, cy - np.sign(cy) * radius
        m = max(2, int(round(0.5 * np.pi * radius / ds)))
        for j in range(m + 1):
            t = (k - 1) * 0.5 * np.pi + 0.5 * np.pi * j / m
            pts.append((cx + radius * np.cos(t), cy + radius * np.sin(t), t))
    out = []
    for (x0, y0, t0), (x1, y1, _) in zip(pts, pts[1:] + pts[:1]):
        out.append((x0, y0, -np.cos(t0), -np.sin(t0)))
        m = int(np.hypot(x1 - x0, y1 - y0) / ds)
        for j in range(1, m):
            out.append((x0 + (x1 - x0) * j / m, y0 + (y1 - y0) * j / m, -np.cos(t0), -np.sin(t0)))
    return np.array(out, np.float32)


@pytest.mark.parametrize("radius,ds", [(3.0, 0.5), (4.0, 1.0), (6.0, 0.25)])
@pytest.mark.parametrize("max_moves", [1, 2, 5, 7, 64])
def test_tight_corners_and_points_far_off(lib, radius, ds, max_moves):
    rows = _rounded_rectangle(radius, ds)
    W = len(rows)
    rng = np.random.default_rng(int(10 * radius) + max_moves)
    n = 60000
    seg0 = rng.integers(0, W - 1, n)
    at = rows[np.clip(seg0 + rng.integers(-6, 12, n), 0, W - 1)]
    xy = at[:, :2] + at[:, 2:] * rng.uniform(-25.0, 25.0, (n, 1)) + rng.normal(0.0, 0.5, (n, 2))
    xy[:20] = np.nan
    want = _search(lib, rows, W, max_moves, xy, seg0, 0)
    for which in (1, 2):
        got = _search(lib, rows, W, max_moves, xy, seg0, which)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), which
