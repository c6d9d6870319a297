"""Host rules of the library that need no GPU: sizes, placements and launch
shapes, through small C entries compiled against its internal headers."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from paper_1708_08739_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if not os.path.exists(build.LIB):
        build.build()
    out = str(tmp_path_factory.mktemp("rules") / "librules.so")
    libdir = os.path.dirname(build.LIB)
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                    "-x", "hip", os.path.join(HERE, "host_rules.cpp"), "-o", out, "-L", libdir, "-l:libbcd.so",
                    "-Wl,-rpath," + libdir], check=True)
    return C.CDLL(out)


def _arr(a):
    return C.c_void_p(a.ctypes.data)


@pytest.mark.parametrize("n,G,P,cap", [(1 << 20, 64, 2, (1 << 31) + 64 * 64), (1000, 3, 1, 48000), (1000, 4, 2, 32000),
                                       (1 << 20, 63, 1, 1 << 32)])
@pytest.mark.parametrize("k", [1, 64, 65, 192])
def test_level0_slots_stay_in_their_lists(rules, n, G, P, cap, k):
    """Staged sources, heavy ones among them, get distinct slots of their own
    list's region, also where a heavy list begins past 2^32 items."""
    slot = np.zeros(k, dtype=np.uint64)
    bounds = np.zeros((k, 2), dtype=np.uint64)
    rules.staged_slots(C.c_int64(n), G, P, C.c_uint64(cap), C.c_uint32(3), k, _arr(slot), _arr(bounds))
    assert np.all(slot >= bounds[:, 0]) and np.all(slot < bounds[:, 1])
    assert np.unique(slot).size == k
    for b in np.unique(bounds[:, 0]):  # packed from the list's beginning
        mine = np.sort(slot[bounds[:, 0] == b])
        assert np.array_equal(mine, b + np.arange(mine.size, dtype=np.uint64))


def test_long_runs_split_from_their_threshold_on(rules):
    """Runs whose sources times arcs reach 2^31 (2^29 weighted) are dealt in an
    even number of equal batches of whole groups; shorter ones, and runs of one
    group, keep the configured width."""
    per = rules.sources_per_batch
    per.argtypes, per.restype = [C.c_int64, C.c_int, C.c_uint64, C.c_uint64], C.c_uint64
    for weighted, bit in ((0, 31), (1, 29)):
        m = 1 << 19
        ns = 1 << (bit - 19)
        width = 64 * 96
        assert per(m, weighted, ns - 1, width) == width
        assert per(m - 1, weighted, ns, width) == width
        groups = ns // 64
        assert per(m, weighted, ns, width) == 64 * -(-groups // 2)
        assert per(1 << 40, weighted, 64, width) == width
        for n in (65, 200, 6145, 20000, 33358):
            p = per(1 << 26, weighted, n, width)
            batches = -(-n // p)
            assert p % 64 == 0 and p <= width
            assert n <= p or batches % 2 == 0 or -(-n // 64) % 2 == 1, (n, p)


def test_workspace_of_a_lease(rules):
    """A call takes the widest idle workspace, a run's second one the narrowest
    that holds its share, else one to be rebuilt."""
    def take(pool, lo=0, hi=0):
        return rules.leased_width(_arr(np.array(pool, dtype=np.int32)), len(pool), lo, hi)
    assert take([]) == 0
    assert take([96, 9]) == 96 and take([9, 96]) == 96
    assert take([96, 9, 12], 9, 96) == 9 and take([96, 9, 12], 10, 96) == 12
    assert take([96, 9, 12], 13, 96) == 96
    assert take([4, 9], 13, 96) == 9
    assert take([128, 100], 13, 96) == 100 and take([128, 4], 13, 96) == 4


@pytest.mark.parametrize("block", [64, 128, 256, 512])
def test_reach_levels_keep_their_wavefronts_at_every_block_size(rules, block):
    """A reachability level runs the configured shape's wavefronts, 4,096 at
    most, whatever the workgroup size of the other kernels."""
    for mult in (1, 8, 32):
        grid = min(8192, 256 * mult)
        waves = rules.reach_grid(block, grid) * 4
        assert waves == min(4096, grid * block // 64), (block, mult)
    assert rules.reach_grid(64, 1) == 1


def test_reachability_in_one_workgroup(rules):
    """Graphs of few arcs, and of more on deep traversals, are searched by one
    workgroup; large ones and shallow ones of many arcs by a launch per level."""
    def one(n, m, levels):
        return bool(rules.one_workgroup(C.c_int64(n), C.c_int64(m), C.c_int64(levels)))
    assert one(2000, 1 << 15, 0) and one(2000, 1 << 15, 6) and not one(2000, (1 << 15) + 1, 9)
    assert one(180 * 180, 4 * 180 * 179, 16) and not one(180 * 180, 4 * 180 * 179, 8)
    assert one(60000, 60000, 12) and one(65535, 15_000_000, 1000)
    assert not one(65535, 60_000_000, 59) and not one(65536, 100, 6) and not one(1 << 20, 100, 1 << 20)


@pytest.mark.parametrize("n", [100, 1 << 20, 1 << 23, (1 << 23) + 1, 1 << 30])
def test_traversals_copy_the_bitmap_once_or_twice(rules, n):
    """The visited bitmap comes to the host with the first check or once at the
    end: at most twice whatever the depth, once where it is large."""
    f = rules.bitmap_bytes_copied
    f.argtypes, f.restype = [C.c_int64, C.c_int64, C.c_int], C.c_uint64
    size = (n + 31) // 32 * 4
    for levels in (0, 3, 7, 8, 9, 63, 64, 1000):
        for first in (4, 8, 64):
            once = levels < first or size > 1 << 20
            assert f(n, levels, first) == size * (1 if once else 2), (levels, first)


@pytest.mark.parametrize("P,H,block", [(1, 0, 256), (2, 0, 64), (2, 7, 256), (2, 500, 512), (1, 3, 128)])
def test_backward_levels_launch_what_their_items_need(rules, P, H, block):
    """A backward level launches no more than a wavefront per light item and
    part of a heavy one and a thread per mask to clear need, with workgroups for
    both lists, and never more than the configured ones."""
    nw = block // 64
    most = 8192 - 8192 % P
    for light in (0, 1, 5, 64, 1000, 10**6):
        for heavy in ((0, 1, 40, 10**5) if H else (0,)):
            for clear in (0, 1, 3000, 10**7):
                cnt = np.zeros(2 * P, dtype=np.uint32)
                cl = np.zeros(2 * P, dtype=np.uint32)
                cnt[P - 1], cnt[2 * P - 1], cl[0] = light, heavy, clear
                a, b = C.c_int(), C.c_int()
                g = rules.bwd_grid(P, C.c_uint32(H), block, most, _arr(cnt), _arr(cl) if clear else None,
                                   C.byref(a), C.byref(b))
                assert g % P == 0 and 2 * P <= g <= most
                if g < most:
                    assert a.value * nw >= light and (heavy == 0 or b.value * nw >= 8 * heavy)
                    assert g // P * block >= clear
                    need = max(2, 1.5 * (light / nw + 1) + 2, 3 * (8 * heavy / nw + 1) + 3 if heavy else 0, clear / block + 1)
                    assert g // P <= need, (light, heavy, clear)


@pytest.mark.parametrize("weighted", [0, 1])
@pytest.mark.parametrize("push,items", [(0, 1), (0, 2), (1, 2), (1, 4)])
def test_autotuner_times_no_setting_twice(rules, weighted, push, items):
    """The candidates around the best one differ from it and from each other in
    something the kernels read; the pushed form is tried at each items value."""
    from paper_1708_08739_amd import bcd
    base = bcd.Config(engine=0, groups=8, block=64 if weighted else 256, grid_mult=32, items=items, bottom_up=0, compress=0,
                      push=0 if weighted else push)
    out = (bcd.Config * 32)()
    k = rules.tune_candidates(C.byref(base), weighted, out, 32)

    def read(c):
        what = (c.engine, c.groups, c.block, c.grid_mult)
        return what if weighted else what + (c.bottom_up, c.push, c.items if c.push else 0)
    seen = [read(c) for c in list(out)[:k]] + [read(base)]
    assert len(set(seen)) == k + 1
    if not weighted:
        assert {s[-1] for s in seen if s[-2] == 1 and s[4] == 0 and s[2] == 256} == {1, 2, 4}
        assert any(s[-2] == 0 for s in seen) and {s[4] for s in seen} == {0, 4, 16}


@pytest.mark.parametrize("stored,c", [(4, 4), (8, 8), (0, 8)])
def test_profile_charges_path_counts_as_stored(rules, stored, c):
    """Bytes of the kernel profile: 4 per path count where rows hold 32 bits,
    8 where they hold 64 (and in the engines that have no narrow rows)."""
    ctr = np.zeros(16, dtype=np.uint64)
    fv, fa, fd, bv, ba, bd = 1000, 20000, 3000, 700, 11000, 900
    ctr[:6] = fv, fa, fd, bv, ba, bd
    ctr[12:] = 50, 800, 40, 600  # items and their arcs, forward and backward
    alg, sched = np.zeros(2), np.zeros(2)
    rules.profile_bytes(stored, _arr(ctr), _arr(alg), _arr(sched))
    assert alg.tolist() == [(24 + c) * fv + 8 * fa + c * fd, (24 + c) * bv + 8 * ba + 8 * bd]
    assert sched.tolist() == [16 * 50 + 4 * 800 + (8 + c) * fv + 4 * fa + c * fd,
                              16 * 40 + 4 * 600 + (8 + c) * bv + 4 * ba + 8 * bd]


@pytest.mark.parametrize("n,m,G", [(1 << 20, 1 << 24, 64), (4097, 50_000, 3), (1 << 18, 1 << 22, 5)])
def test_workspace_bytes_count_the_heavy_lists(rules, n, m, G):
    """The bytes a server's budget is checked against hold the heavy vertices'
    item lists (64 items of 12 bytes a group) and queue entries (4 of 4 bytes),
    and every per-level and per-vertex array."""
    f = rules.workspace_bytes
    f.argtypes, f.restype = [C.c_int64, C.c_int64, C.c_uint32, C.c_int, C.c_int], C.c_uint64
    H = n // 256
    assert f(n, m, H, 0, G) - f(n, m, 0, 0, G) >= G * H * 64 * 12
    assert f(n, m, H, 1, G) - f(n, m, 0, 1, G) >= G * H * (64 * 12 + 16)
    rows = G * n * 64 * 16 + G * n * 16 * 12 + 4 * n * 12 + 4 * n
    assert rows + 72 * G * n <= f(n, m, 0, 0, G) <= rows + 72 * G * n + (4 << 20)
    assert rows + G * n * (64 * 8 + 64 + 16) + 8 * G * m <= f(n, m, 0, 1, G)


def test_lds_engine_takes_short_rows_alone(rules):
    """The LDS engine takes arcs one at a time where no row has more than two."""
    assert [rules.short_rows(C.c_int64(k)) for k in (0, 1, 2, 3, 4, 5000)] == [1, 1, 1, 0, 0, 0]


@pytest.mark.parametrize("weighted,m", [(1, 3938872), (0, 16085068), (0, 1000)])
def test_timed_samples_take_the_second_workspace_of_their_run(rules, weighted, m):
    """A run's second workspace holds one of its batches.  A sample that the
    autotuner times in its place takes one as wide as the run's (its own batches
    can be narrower), so a width whose pair the device cannot hold is timed on one
    workspace, as it would run; a run of one batch takes none."""
    f, per = rules.second_workspace_groups, rules.sources_per_batch
    f.argtypes, f.restype = [C.c_int64, C.c_int, C.c_uint64, C.c_uint64, C.c_uint64], C.c_int
    per.argtypes, per.restype = [C.c_int64, C.c_int, C.c_uint64, C.c_uint64], C.c_uint64
    for groups in (1, 3, 16, 128, 256):
        width = 64 * groups
        for ns in (1, 64, 65, 2048, 16384, 150000):
            own = per(m, weighted, ns, width)
            alone = 0 if ns <= own else -(-own // 64)
            assert f(m, weighted, ns, 0, width) == alone
            assert f(m, weighted, ns, ns, width) == alone
            for whole in (ns + 1, 130 * 64, 150000):
                if whole < ns:
                    continue
                want = max(own, per(m, weighted, whole, width))
                assert f(m, weighted, ns, whole, width) == (-(-want // 64) if ns > own else 0)
    # 16,384 of 150,000 sources at 256 groups: two batches of 128 groups, the run's ten have 235
    if weighted:
        assert f(m, 1, 16384, 0, 16384) == 128 and f(m, 1, 16384, 150000, 16384) == -(-2344 // 10)
