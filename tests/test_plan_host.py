"""The device planner compiled for the host (tests/host_plan) under AddressSanitizer.

* Inconsistent grouping arrays, including group sizes whose 32-bit sum wraps around to
  n_suffixes, are flagged and never make the planner read past an array.
* Valid arrays: the one-block and the multi-kernel planners give the same plan for every
  tiling the library runs, and the plan is what the kernels assume (prefix tiles of every group, response rows of
  every group stacked into tiles, per-tile member bounds, longest-first order).
* Every load the attention kernels derive from the plan (key/value tiles of the forward
  and dQ kernels, query tiles of the dK/dV walks, per-row tables) stays inside its tensor
  and inside a 2^31-byte buffer range, for the five workloads and the Fig. 2/3 grid.
"""
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2506_05433_amd.inputs import WORKLOADS, Workload, draw_lengths

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host_plan")
CSRC = os.path.join(ROOT, "paper_2506_05433_amd", "csrc")
BN = {128: 64, 256: 32}  # keys per staged tile, by the query rows of a workgroup
BQ = {"bf16": 64, "fp32": 32}  # query rows per staged tile of the 128-key dK/dV kernel; 32 for 256 keys
DTYPES = {"bf16": 0, "fp32": 1}
TILINGS = [(0, 0), (1, 0), (1, 1)]  # 128 rows and keys, 128 rows and 256 keys, 256 rows and keys


def build_planner(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("plan") / "plan_host")
    cmd = [gxx, "-std=c++20", "-O1", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
           "-fno-sanitize-recover=undefined", "-pthread", "-I", HERE, "-I", CSRC,
           os.path.join(HERE, "plan_host.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return exe


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    return build_planner(tmp_path_factory)


def layouts(exe, calls):
    """The library's choices (pg_layout.hpp) for backward calls (dtype, ng, ns, tp, ts, h_q, h_kv, d) or, with two
    more values, for a given tiling (wide, wide_q)."""
    keys = ("bm", "bkv", "kvc", "split", "max_q", "max_kv", "one_block", "workspace", "size_query")
    text = "2\n" + "\n".join(" ".join(str(int(x)) for x in (tuple(c) + (-1, -1))[:10]) for c in calls)
    res = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stderr[-4000:]
    return [dict(zip(keys, map(int, line.split()))) for line in res.stdout.strip().split("\n")]


def bounds(ng, ns, tp, ts, kvc, bm, bkv):
    return (math.ceil(tp / bm) + math.ceil(ts / bm) + 2 * ng + ns,
            (math.ceil(tp / bkv) + ng) * kvc + math.ceil(ts / bkv) + ng + ns)


def run_plan(exe, cu_p, cu_s, gsz, ng, ns, tp, ts, mode=0, kvc=1, split=0, max_q=None, max_kv=None, bm=128, bkv=128):
    bq, bk = bounds(ng, ns, tp, ts, kvc, bm, bkv)
    max_q = bq if max_q is None else max_q
    max_kv = bk if max_kv is None else max_kv
    lines = _run(exe, [mode, ng, ns, tp, ts, bm, bkv, kvc, split, max_q, max_kv, *cu_p, *cu_s, *gsz])
    err, nq, nkv = (int(x) for x in lines[0].split())
    q = [tuple(int(x) for x in ln.split()[1:]) for ln in lines[1:] if ln.startswith("q ")]
    k = [tuple(int(x) for x in ln.split()[1:]) for ln in lines[1:] if ln.startswith("k ")]
    s = [ln for ln in lines if ln.startswith("s")]
    seg = [int(x) for x in s[0].split()[1:]] if s else []
    return err, q, k, seg


def run_last_plan(exe, cu_p, cu_s, gsz, ng, ns, tp, ts, mpw, nb_max, mode):
    """(error, member blocks) of the final-token call's plan: mode 3 in one kernel, 4 in two."""
    lines = _run(exe, [mode, ng, ns, tp, ts, mpw, nb_max, *cu_p, *cu_s, *gsz])
    err, n = (int(x) for x in lines[0].split())
    blocks = [tuple(int(x) for x in ln.split()[1:]) for ln in lines[1:] if ln.startswith("b ")]
    assert len(blocks) == n
    return err, blocks


def _run(exe, values):
    text = " ".join(str(int(x)) for x in values)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0", UBSAN_OPTIONS="halt_on_error=1")
    res = subprocess.run([exe], input=text, capture_output=True, text=True, env=env, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    assert "ERROR: AddressSanitizer" not in res.stderr and "runtime error" not in res.stderr, res.stderr[-4000:]
    return res.stdout.split("\n")


def arrays(prefix, groups, suffix):
    cu_p = np.concatenate([[0], np.cumsum(prefix)]).astype(np.int64)
    cu_s = np.concatenate([[0], np.cumsum(suffix)]).astype(np.int64)
    return cu_p, cu_s, np.asarray(groups, np.int64)


def test_workspace_query_is_what_one_of_the_types_needs(planner):
    """pg_attn_bwd_workspace_size is the larger of the two types' needs, and the 128-key layout alone where no
    type takes the 256-key kernel: 17 groups of 1000 rows (whose size a second tiling raised from 3 to 274 MB)."""
    rng = np.random.default_rng(11)
    calls = [(17, 68, 17000, 4096, 32, 8, 128)]
    for _ in range(300):
        h_kv = int(rng.choice([1, 2, 4, 8]))
        ng = int(rng.integers(1, 20))
        calls.append((ng, ng * int(rng.integers(0, 20)), int(10 ** rng.uniform(0, 5)), int(10 ** rng.uniform(0, 5.3)),
                      h_kv * int(rng.choice([1, 4, 8])), h_kv, int(rng.choice([64, 128]))))
    bf16, fp32 = (layouts(planner, [(t, *c) for c in calls]) for t in (0, 1))
    narrow = layouts(planner, [(0, *c, 0, 0) for c in calls])
    assert {lay["bkv"] for lay in bf16} == {128, 256} and all(lay["bkv"] == 128 for lay in fp32)
    for a, b, n in zip(bf16, fp32, narrow):
        assert a["size_query"] == b["size_query"] == max(a["workspace"], b["workspace"])
        assert a["bkv"] == 256 or a["size_query"] == n["workspace"]
    assert bf16[0]["bkv"] == 128


@pytest.mark.parametrize("ng,ns,tp,ts,h_q,h_kv,d,pieces", [
    # (sizes, pieces of a prefix walk with 256-key tiles): on both sides of each line of kv_chunks_wide
    (1, 8, 13367, 1407, 8, 2, 128, 4),
    (1, 8, 4096, 5120, 32, 8, 128, 3),
    (3, 6, 24635, 657, 16, 4, 128, 2),      # 388..400 tiles
    (1, 16, 16384, 5120, 32, 8, 128, 1),    # 512: two whole rounds
    (2, 32, 17576, 7824, 40, 8, 128, 2),    # 552..568: just above them
    (2, 6, 22928, 224, 40, 8, 128, 1),      # 720
    (7, 434, 13080, 20622, 8, 8, 128, 1),   # one query head per kv head: short walks, cut in two they ran 20% longer
    (10, 100, 40758, 3595, 4, 4, 128, 1),   # the same, 30%
    (6, 66, 30268, 4338, 2, 2, 128, 2),     # short walks, but fewer tiles than CUs
])
def test_pieces_of_the_256_key_walks(planner, ng, ns, tp, ts, h_q, h_kv, d, pieces):
    (lay,) = layouts(planner, [(0, ng, ns, tp, ts, h_q, h_kv, d, 1, 0)])
    assert lay["kvc"] == pieces and lay["bkv"] == 256


@pytest.mark.parametrize("ng,ns,tp,ts,h_q,h_kv,d,keys", [
    # on both sides of each line of use_wide
    (1, 52, 2440, 17456, 5, 1, 128, 128),   # 10 tiles, eight pieces each: 334 us, with 256 keys 515
    (1, 53, 7653, 2290, 8, 1, 64, 128),     # 30 tiles: 249, 320
    (1, 55, 12122, 1742, 8, 1, 128, 256),   # 48 tiles: 846, 697
    (17, 68, 17000, 4096, 32, 8, 128, 128),  # prefixes of 1000 rows
    (9, 72, 13059, 29013, 32, 8, 128, 256),  # of 1451
    (1, 5, 1024, 1000, 32, 8, 128, 128),    # 24 steps per CU
    (1, 8, 2048, 5120, 32, 8, 128, 256),
])
def test_choice_of_the_256_key_kernel(planner, ng, ns, tp, ts, h_q, h_kv, d, keys):
    (lay,) = layouts(planner, [(0, ng, ns, tp, ts, h_q, h_kv, d)])
    assert lay["bkv"] == keys


@pytest.mark.parametrize("gsz,ns", [
    # 32-bit sums that wrap around to n_suffixes (the planner would then index cu_suffix_lens with
    # member starts near 2^31)
    ([0x7FFFFFFF, 0x7FFFFFFF, 2], 0),
    ([0x7FFFFFFF, 0x7FFFFFFF, 5], 3),
    ([0x40000000] * 4 + [3], 3),
    ([-1, 4], 3),
    ([5, 1], 3),
])
def test_inconsistent_group_sizes_are_flagged_without_out_of_range_reads(planner, gsz, ns):
    ng = len(gsz)
    cu_p = list(range(ng + 1))          # one prefix row per group: valid
    cu_s = list(range(ns + 1))          # one row per member: valid
    _all_planners_refuse(planner, cu_p, cu_s, gsz, ng, ns)


def _all_planners_refuse(planner, cu_p, cu_s, gsz, tp, ts):
    """The arrays are flagged: as they are, planned from LDS, and padded with empty groups (in front, so that the
    fault sits beyond the first pass of 1024) or members to more than LDS holds (plan_groups_kernel from memory, here
    before plan_last_kernel)."""
    ng, ns = len(gsz), len(cu_s) - 1
    for mode in (0, 1):
        err, q, k, _ = run_plan(planner, cu_p, cu_s, gsz, ng, ns, tp, ts, mode=mode)
        assert err == 1 and not q and not k
    assert run_last_plan(planner, cu_p, cu_s, gsz, ng, ns, tp, ts, 16, ns + ng, 3) == (1, [])
    more_groups = ([cu_p[0]] * 1100 + list(cu_p), list(cu_s), [0] * 1100 + list(gsz))
    more_members = (list(cu_p), list(cu_s) + [cu_s[-1]] * 4097, list(gsz[:-1]) + [gsz[-1] + 4097])
    if gsz[-1] + 4097 > 0x7FFFFFFF or gsz[-1] < 0:
        more_members = None
    for a in filter(None, (more_groups, more_members)):
        n, m = len(a[2]), len(a[1]) - 1
        assert run_last_plan(planner, *a, n, m, tp, ts, 16, m + n, 4) == (1, [])


@pytest.mark.parametrize("bad", ["cu_p_start", "cu_p_total", "cu_p_order", "cu_s_total", "cu_s_order", "size_sum"])
def test_inconsistent_offsets_are_flagged(planner, bad):
    cu_p, cu_s, gsz = (list(a) for a in arrays([5, 3], [2, 1], [4, 0, 6]))
    tp, ts = 8, 10
    if bad == "cu_p_start":
        cu_p[0] = 1
    elif bad == "cu_p_total":
        tp = 9
    elif bad == "cu_p_order":
        cu_p[1] = 9
    elif bad == "cu_s_total":
        ts = 11
    elif bad == "cu_s_order":
        cu_s[1] = 7
    else:
        gsz = [2, 2]
    _all_planners_refuse(planner, cu_p, cu_s, gsz, tp, ts)


@pytest.mark.parametrize("ng,mpw", [(1, 16), (7, 2), (63, 16), (64, 1), (300, 3), (1023, 2), (1024, 2), (2500, 1)])
def test_member_blocks_of_the_final_token_plan(planner, ng, mpw):
    """Every group's members in runs of at most mpw, groups in order; both ways of planning where both apply."""
    rng = np.random.default_rng(ng)
    groups = rng.integers(0, 5, ng) if ng > 1 else np.array([40])
    suffix = rng.integers(0, 9, int(groups.sum()))
    prefix = rng.integers(0, 9, ng)
    cu_p, cu_s, gsz = arrays(prefix, groups, suffix)
    ns = len(suffix)
    want, m = [], 0
    for g, size in enumerate(groups):
        want += [(g, m + i, min(mpw, int(size) - i)) for i in range(0, int(size), mpw)]
        m += int(size)
    modes = (3, 4) if ng <= 1023 and ns <= 4096 else (4,)
    for mode in modes:
        assert run_last_plan(planner, cu_p, cu_s, gsz, ng, ns, cu_p[-1], cu_s[-1], mpw, ns + ng, mode) == (0, want)


def expected_tiles(prefix, groups, suffix, kvc, split=0, bm=128, bkv=128):
    """The tiling the kernels assume, as sets of (kind, group, row0, row1, aux, chunk, nchunks): prefix tiles
    of every group; response rows of a group stacked into tiles across member boundaries, or with ``split``
    each member's rows tiled on their own."""
    cu_p, cu_s, _ = arrays(prefix, groups, suffix)
    q, k = set(), set()
    m = 0
    for g, (p, gs) in enumerate(zip(prefix, groups)):
        p0, p1 = int(cu_p[g]), int(cu_p[g + 1])
        spans = ([(int(cu_s[i]), int(cu_s[i + 1])) for i in range(m, m + gs)] if split
                 else [(int(cu_s[m]), int(cu_s[m + gs]))])
        owner = lambda row: int(np.searchsorted(cu_s, row, side="right") - 1)  # noqa: E731
        for r0 in range(p0, p1, bm):
            q.add((0, g, r0, min(r0 + bm, p1), 0, 0, 1))
        for r0 in range(p0, p1, bkv):
            for c in range(kvc):
                k.add((0, g, r0, min(r0 + bkv, p1), 0, c, kvc))
        for s0, s1 in spans:
            for r0 in range(s0, s1, bm):
                q.add((1, g, r0, min(r0 + bm, s1), int(cu_s[owner(r0)]), 0, 1))
            for r0 in range(s0, s1, bkv):
                r1 = min(r0 + bkv, s1)
                k.add((1, g, r0, r1, int(cu_s[owner(r1 - 1) + 1]), 0, 1))
        m += gs
    return q, k


def check_loads(prefix, groups, suffix, q, k, seg, h_q, h_kv, d, dtype, bm=128, bkv=128):
    """Every tensor row range the kernels load from a planned tile lies inside its tensor, and every
    buffer range (valid rows of one staged tile x row bytes) stays below 2^31 bytes."""
    cu_p, cu_s, _ = arrays(prefix, groups, suffix)
    tp, ts = int(cu_p[-1]), int(cu_s[-1])
    el = 2 if dtype == "bf16" else 4
    bq, bn = BQ[dtype] if bkv == 128 else 32, BN[bm]
    gm = np.concatenate([[0], np.cumsum(groups)]).astype(np.int64)
    rng_pre = {g: (int(cu_p[g]), int(cu_p[g + 1])) for g in range(len(prefix))}
    rng_suf = {g: (int(cu_s[gm[g]]), int(cu_s[gm[g + 1]])) for g in range(len(prefix))}
    assert seg == cu_s[np.searchsorted(cu_s, np.arange(ts), side="right") - 1].tolist()

    def rows_ok(lo, hi, n, what):
        assert 0 <= lo < hi <= n, (what, lo, hi, n)

    for (kind, g, row0, row1, aux, work, chunk, nch) in q:
        p0, p1 = rng_pre[g]
        # the tile's own query rows (loaded row by row, clamped to row1 - 1)
        rows_ok(row0, row1, ts if kind else tp, "query rows")
        segs = [(p0, row1 if kind == 0 else p1, tp)] + ([(aux, row1, ts)] if kind else [])
        for lo, hi, n in segs:
            for k0 in range(lo, hi, bn):
                valid = min(bn, hi - k0)
                rows_ok(k0, k0 + valid, n, "key tile")
                assert valid * h_kv * d * el < 2 ** 31
        if kind:
            assert rng_suf[g][0] <= aux <= row0
    for (kind, g, row0, row1, aux, work, chunk, nch) in k:
        p0, p1 = rng_pre[g]
        s0, s1 = rng_suf[g]
        rows_ok(row0, row1, ts if kind else tp, "key rows")
        ranges = [(s0, s1, ts), (row0, p1, tp)] if kind == 0 else [(row0, aux, ts)]
        for lo, hi, n in ranges:
            for q0 in range(lo, hi, bq):
                valid = min(bq, hi - q0)
                rows_ok(q0, q0 + valid, n, "query tile")
                assert valid * h_q * d * el < 2 ** 31


def _planned(planner, prefix, groups, suffix, h_q, h_kv, d=128, dtype="bf16", tiling=(-1, -1), modes=(0, 1),
             split=None):
    """Plans of the one-block planner (only where the library uses it: both tile lists within one block)
    and of the multi-kernel planner, for the library's layout of these sizes or a given tiling; modes=None: the
    planner the library would run. ``split`` defaults to the library's choice."""
    cu_p, cu_s, gsz = arrays(prefix, groups, suffix)
    ng, ns, tp, ts = len(prefix), len(suffix), int(cu_p[-1]), int(cu_s[-1])
    (lay,) = layouts(planner, [(DTYPES[dtype], ng, ns, tp, ts, h_q, h_kv, d, *tiling)])
    if split is not None:
        lay["split"] = split
    if modes is None:
        modes = (0,) if lay["one_block"] else (1,)
    plans = [run_plan(planner, cu_p, cu_s, gsz, ng, ns, tp, ts, mode=mode, **{k: lay[k] for k in (
        "kvc", "split", "max_q", "max_kv", "bm", "bkv")}) for mode in modes if mode == 1 or lay["one_block"]]
    return plans, lay


@pytest.mark.parametrize("tiling", TILINGS)
@pytest.mark.parametrize("seed,split", [(s, s % 2) for s in range(6)])
def test_random_groupings_plan_as_the_kernels_assume(planner, seed, split, tiling):
    rng = np.random.default_rng(seed)
    ng = int(rng.integers(1, 40))
    prefix = rng.integers(0, 600, ng) * (rng.random(ng) < 0.8)
    groups = rng.integers(0, 6, ng)
    suffix = rng.integers(0, 400, int(groups.sum())) * (rng.random(int(groups.sum())) < 0.9)
    (fused, multi), lay = _planned(planner, prefix, groups, suffix, 8, 2, tiling=tiling, split=split)
    assert fused == multi and (lay["bm"], lay["bkv"]) == (128 << tiling[1], 128 << tiling[0])
    err, q, k, seg = fused
    assert err == 0
    eq, ek = expected_tiles(list(prefix), list(groups), list(suffix), lay["kvc"], split, lay["bm"], lay["bkv"])
    assert set(t[:5] + t[6:] for t in q) == eq and len(q) == len(eq)
    assert set(t[:5] + t[6:] for t in k) == ek and len(k) == len(ek)
    for tiles in (q, k):
        work = [t[5] for t in tiles]
        assert work == sorted(work, reverse=True)
    check_loads(prefix, groups, suffix, q, k, seg, 8, 2, 128, "bf16", lay["bm"], lay["bkv"])


@pytest.mark.parametrize("pad", ["groups", "members"])
def test_plan_from_memory_is_the_plan_from_lds(planner, pad):
    """Empty groups or members behind the others, more than LDS holds, change no tile."""
    rng = np.random.default_rng(21)
    prefix, groups = rng.integers(0, 500, 40), rng.integers(0, 5, 40)
    suffix = rng.integers(0, 300, int(groups.sum()))
    cu_p, cu_s, gsz = (list(a) for a in arrays(prefix, groups, suffix))
    plans = []
    for extra in (0, 1100 if pad == "groups" else 4097):
        if pad == "groups":
            a = (cu_p + cu_p[-1:] * extra, cu_s, gsz + [0] * extra)
        else:
            a = (cu_p, cu_s + cu_s[-1:] * extra, gsz[:-1] + [gsz[-1] + extra])
        plans.append(run_plan(planner, *a, len(a[2]), len(a[1]) - 1, cu_p[-1], cu_s[-1], mode=1))
    assert plans[0] == plans[1] and plans[0][0] == 0


@pytest.mark.parametrize("ng", [1, 62, 63, 64, 65, 128, 500])
def test_group_counts_around_a_wave(planner, ng):
    """The prefix sums over groups within one wave, and from one wave to the next."""
    rng = np.random.default_rng(ng)
    prefix, groups = rng.integers(0, 300, ng), rng.integers(0, 3, ng)
    suffix = rng.integers(0, 200, int(groups.sum()))
    plans, lay = _planned(planner, prefix, groups, suffix, 4, 4, split=0)
    assert (len(plans) == 2) == (ng <= 128)
    eq, ek = expected_tiles(list(prefix), list(groups), list(suffix), lay["kvc"])
    for err, q, k, _ in plans:
        assert err == 0 and set(t[:5] + t[6:] for t in q) == eq and len(q) == len(eq)
        assert set(t[:5] + t[6:] for t in k) == ek and len(k) == len(ek)


@pytest.mark.parametrize("name", ["tiny", "single_group", "long_prefix", "large_group", "packed_varlen"])
def test_workload_loads_stay_in_range(planner, name):
    """With the library's own tiling and with the others its kernels take."""
    wl = WORKLOADS[name]
    prefix, groups, suffix = draw_lengths(wl, 0)
    own = None
    for tiling in [(-1, -1)] + (TILINGS if wl.dtype == "bf16" else []):
        plans, lay = _planned(planner, prefix, groups, suffix, wl.h_q, wl.h_kv, wl.head_dim, wl.dtype, tiling)
        if tiling == (-1, -1):
            own = lay
        elif lay == own:
            continue
        assert all(p == plans[0] for p in plans) and plans[0][0] == 0
        _, q, k, seg = plans[0]
        check_loads(prefix, groups, suffix, q, k, seg, wl.h_q, wl.h_kv, wl.head_dim, wl.dtype, lay["bm"], lay["bkv"])


def test_fig23_grid_loads_stay_in_range(planner):
    """Corners of the bench sweep's grid (P 4096/16384, G 2/16, responses around P/r for r = 1, 16; the
    middle points plan the same way), plus the 2 GiB dense query range that once overran its buffer
    (16 members of 1024 rows at h_q * d = 65536)."""
    for P in (4096, 16384):
        for G in (2, 16):
            for r in (1, 16):
                S = P // r
                wl = Workload("grid", 1, G, ("fixed", P), ("uniform", S // 2, S + S // 2), 32, 8, 128, "bf16", 1.0)
                prefix, groups, suffix = draw_lengths(wl, 0)
                (plan,), lay = _planned(planner, prefix, groups, suffix, 32, 8, modes=None)
                check_loads(prefix, groups, suffix, plan[1], plan[2], plan[3], 32, 8, 128, "bf16", lay["bm"], lay["bkv"])
    prefix, groups, suffix = [128], [16], [1024] * 16
    (plan,), lay = _planned(planner, prefix, groups, suffix, 512, 64, modes=None)
    check_loads(prefix, groups, suffix, plan[1], plan[2], plan[3], 512, 64, 128, "bf16", lay["bm"], lay["bkv"])
