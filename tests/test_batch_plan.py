"""The batch planner on the host: csrc/plan.cpp built on its own, with a table
of the work-groups a device of 256 CUs holds in place of the runtime's query.

Members that the autotuner has left with a rule's tiles plan to the layout that
it timed under the rule, so that one fits a workspace sized for all rules.  The
chunk length is the one that the model's least time over all lengths gives.
"""
import ctypes as C
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2501_02317_amd", "csrc")
RULES = 12

HARNESS = r"""
#include <algorithm>
#include "plan.h"
using namespace hydro;
static Slots residency(int ndim, int precision, int mode, const Tile& t) {
    const int waves = (t.tx * t.ty + 63) / 64;
    return {256, (ndim == 3 && precision == 0 ? 12 : 16) / waves, waves};
}
// The model of auto_kz over every length and every column by itself.
static int every_kz(int ndim, const Slots& sl, const MarchCols* m, int n, double* time) {
    int most = 1;
    for (int i = 0; i < n; ++i) most = std::max(most, m[i].n2);
    most = std::min(most, kMaxAutoKz);
    const double lead = ndim == 3 ? 2.0 : 3.0;
    const long long slots = (long long)sl.cus * sl.per_cu;
    auto plane = [&](long long wgs) {
        const double w = (double)((wgs + sl.cus - 1) / sl.cus) * sl.waves / 4.0;
        return w > 1.0 ? 1.0 + (w - 1.0) / 3.0 : 1.0;
    };
    int best = most;
    for (int kz = most; kz >= 1; --kz) {
        long long wgs = 0;
        for (int i = 0; i < n; ++i) wgs += m[i].cols * ((m[i].n2 + kz - 1) / kz);
        const long long full = wgs / slots, rest = wgs % slots;
        double t = (kz + lead) * (full * plane(slots) + (rest ? plane(rest) : 0.0));
        if (n == 1 && m[0].per_xcd && full == 1 && rest > 0 && 2 * slots + m[0].cols >= 2 * wgs) {
            const int last = m[0].n2 - (m[0].n2 - 1) / kz * kz;
            t = std::min(t, plane(slots) * std::max(kz + lead, 2.0 * (last + lead)));
        }
        if (kz == most || t <= *time) {
            *time = t;
            best = kz;
        }
    }
    return best;
}
// q: (columns, n2) each; whether auto_kz finds the same length and time.
extern "C" int same_kz(int ndim, int per_cu, int waves, int n, const int* q, int per_xcd) {
    std::vector<MarchCols> m;
    for (int i = 0; i < n; ++i) m.push_back({q[2 * i], q[2 * i + 1], per_xcd != 0});
    double a = 0.0, b = 0.0;
    const Slots sl{256, per_cu, waves};
    const int ka = auto_kz(ndim, sl, m.data(), n, &a), kb = every_kz(ndim, sl, m.data(), n, &b);
    return ka == kb && a == b;
}
extern "C" int default_shape(int ndim, int precision, int n0, int n1, int n2) {
    Geo g{};
    g.ndim = ndim;
    g.n[0] = n0;
    g.n[1] = n1;
    g.n[2] = n2;
    const Tile t = default_tile(g, precision, MODE_STAGE1);
    return 1000 * t.tx + t.ty;
}
// members: (ndim, precision, integrator, n0, n1, n2, tx, ty, kz) each, tx 0: the default tile.
// out: work-groups, groups, then per member (in descriptor order) its index, tiles and chunks.
extern "C" int plan(int n, const int* q, int rule, int tuned, int* out) {
    std::vector<PlanMember> m(n);
    for (int i = 0; i < n; ++i, q += 9) {
        Geo& g = m[i].geo;
        g = Geo{};
        g.ndim = q[0];
        g.n[0] = q[3];
        g.n[1] = q[4];
        g.n[2] = q[5];
        g.ncells = (long long)q[3] * q[4] * q[5];
        for (int k = 0; k < 3; ++k) g.blocks[k] = 1;
        m[i].precision = q[1];
        m[i].integrator = q[2];
        m[i].tile_set = q[6] > 0;
        m[i].tile = q[6] > 0 ? Tile{q[6], q[7], q[8]} : default_tile(g, q[1], q[2] ? MODE_VL2_PRED : MODE_STAGE1);
    }
    // the tiles that the autotuner leaves when the rule has won
    for (int i = 0; i < n && tuned && rule > 0; ++i)
        if (m[i].geo.ndim < 3) {
            m[i].tile = rule_tile(m[i], rule);
            m[i].tile_set = true;
        }
    BatchLayout L;
    if (!plan_layout(m, tuned ? 0 : rule, residency, L)) return -1;
    *out++ = L.nblk;
    *out++ = (int)L.groups.size();
    for (int i : L.order) {
        const MemberTiling& t = L.tiling[i];
        *out++ = i;
        *out++ = t.tiles_x;
        *out++ = t.tiles_y;
        *out++ = t.chunks_z;
        *out++ = t.kz;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src = d / "harness.cpp"
    src.write_text(HARNESS)
    out = d / "libplan.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    str(src), os.path.join(CSRC, "plan.cpp"), "-o", str(out)], check=True)
    return C.CDLL(str(out))


def plan(lib, members, rule, tuned=False):
    n = len(members)
    q = (C.c_int * (9 * n))(*[v for m in members for v in m])
    out = (C.c_int * (2 + 5 * n))()
    assert lib.plan(n, q, rule, int(tuned), out) == 0
    return list(out)


def member(n, precision=1, integrator=0, tile=(0, 0, 0)):
    nd = len(n)
    k = {1: (n[0], 1, 1), 2: (n[0], 1, n[-1]), 3: n}[nd]
    return (nd, precision, integrator, *k, *tile)


def mixes():
    """2-D and 3-D requests as a server admits them, among them members whose
    tile was set."""
    rng = random.Random(5)
    yield [member((a,) * 3) for a in (144, 160, 32, 80, 144)] + [member((a,) * 2) for a in (448, 352, 992, 416, 832)]
    for _ in range(150):
        m = []
        for _ in range(rng.randint(2, 14)):
            p, i, kind = rng.randint(0, 1), rng.choice([0, 0, 0, 1]), rng.random()
            if kind < 0.45:
                n = (16 * rng.randint(2, 10),) * 3
                m.append(member(n, p, i, rng.choice([(0, 0, 0)] * 4 + [(16, 16, 0), (32, 8, 3)])))
            elif kind < 0.95:
                n = (32 * rng.randint(2, 32),) * 2
                m.append(member(n, p, i, rng.choice([(0, 0, 0)] * 4 + [(64, 1, 0), (256, 1, 2)])))
            else:
                m.append(member((64 * rng.randint(1, 40),), p, i))
        yield m


def test_tuned_layout_is_the_timed_one_and_fits(lib):
    for m in mixes():
        rules = [plan(lib, m, r) for r in range(RULES)]
        most = max(p[0] for p in rules)
        for r in range(RULES):
            got = plan(lib, m, r, tuned=True)
            assert got[0] <= most, (m, r, got[0], most)
            assert got == rules[r], (m, r)


def test_default_tiles_are_shared(lib):
    """Ragged 2-D meshes and cubes of both default widths: one launch for each
    dimensionality, where each member's own tile would make five."""
    m = [member(n) for n in [(64,) * 2, (96,) * 2, (200, 160), (384, 100), (512,) * 2, (48,) * 3, (64,) * 3]]
    # rows of 64, 128 and 256; 16 x 16 and 32 x 16
    assert len({(q[0], lib.default_shape(q[0], q[1], *q[3:6])) for q in m}) == 5
    assert plan(lib, m, 0)[1] == 2


def test_chunk_length_has_the_least_modelled_time(lib):
    rng = random.Random(8)
    for i in range(3000):
        n = rng.choice([1, 1, 2, 5])
        q = [v for _ in range(n) for v in (int(2 ** rng.uniform(0, 13)), int(2 ** rng.uniform(0, 11)))]
        waves = rng.choice([1, 2, 4, 8])
        args = (rng.choice([2, 3]), rng.choice([1, 2, 3, 4, 16 // waves]), waves, n, (C.c_int * len(q))(*q), i % 3 == 0)
        assert lib.same_kz(*args), (q, args)
