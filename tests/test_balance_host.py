"""Host check of how the FFT launches share their templates out over workgroups (csrc/balance.cpp).

The rule is arithmetic on counts, compiled here without HIP. An independent dispatch (each tile in
turn to the place that is free first, one heap operation a tile) says what the plan's own blocks
and the chosen ones take: a tile costs its templates and a forward transform worth 1.5 of them.
"""

import ctypes
import heapq
import os
import random
import subprocess
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1911_01353_amd", "csrc")
PLACES = 2048


class Run(ctypes.Structure):
    _fields_ = [("segs", ctypes.c_int64), ("members", ctypes.c_int32), ("tpb", ctypes.c_int32), ("free", ctypes.c_bool)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("balance")
    src = d / "entry.cpp"
    src.write_text('#include "balance.h"\n'
                   'extern "C" void choose(jerk::BalanceRun* r, int n, int64_t places, int64_t most, bool in_order) {\n'
                   '  jerk::balance_blocks(r, n, places, most, in_order);\n}\n'
                   'extern "C" double finish(const jerk::BalanceRun* r, int n, int64_t places) {\n'
                   '  return jerk::dispatch_time(r, n, places, 1e300);\n}\n'
                   'extern "C" bool allowed(int32_t tpb, int32_t own, int32_t U, double pre) {\n'
                   '  return jerk::candidate_blocks_allowed(tpb, own, U, pre);\n}\n')
    so = d / "libbalance.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src),
                    os.path.join(CSRC, "balance.cpp"), "-o", str(so)], check=True)
    out = ctypes.CDLL(str(so))
    out.choose.argtypes = [ctypes.POINTER(Run), ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_bool]
    out.finish.argtypes = [ctypes.POINTER(Run), ctypes.c_int, ctypes.c_int64]
    out.finish.restype = ctypes.c_double
    out.allowed.argtypes = [ctypes.c_int32, ctypes.c_int32, ctypes.c_int32, ctypes.c_double]
    out.allowed.restype = ctypes.c_bool
    return out


def tiles(runs):
    for r in runs:
        for m0 in range(0, r.members, r.tpb):
            c = min(r.tpb, r.members - m0) + 1.5
            for _ in range(r.segs):
                yield c


def dispatched(runs, places=PLACES):
    busy, end = [0.0] * places, 0.0
    for c in tiles(runs):
        t = heapq.heappop(busy) + c
        heapq.heappush(busy, t)
        end = max(end, t)
    return end


def default_tpb(n_seg, members):
    return next((t for t in (64, 32, 16, 8) if n_seg * -(-members // t) >= 4096), 4)


def launch(rng):
    """The first launch of a search of some rows of a grid, as a default plan lays it out: up to eight
    width groups, narrowest first."""
    zmax = 2 * rng.randint(10, 110)
    wmax = rng.choice([0, 1, 3]) * zmax
    n = int(2 ** rng.uniform(15, 21))
    half = {}
    t = 0
    count = (zmax + 1) * (2 * (wmax // 20) + 1)
    rows = min(count, rng.randint(8, 320))
    t0 = (count - rows) // 2
    whole = {}
    for j in range(-(wmax // 20), wmax // 20 + 1):
        for i in range(zmax + 1):
            h = -(-abs(-zmax + 2 * i) // 2) if not j else int(abs(-zmax + 2 * i) / 2 + abs(20 * j) / 12 + 0.999999)
            taps = (2 * (h + 16) + 15) // 16 * 16
            whole[taps] = whole.get(taps, 0) + 1
            if t0 <= t < t0 + rows:
                half[taps] = half.get(taps, 0) + 1
            t += 1
    out = []
    for taps in sorted(half)[:8]:
        segs = -(-n // (1024 - taps + 1))
        out.append(Run(segs, half[taps], default_tpb(segs, whole[taps]), True))
    return out


def copy(runs):
    return (Run * len(runs))(*[Run(r.segs, r.members, r.tpb, r.free) for r in runs])


def test_dispatch_time_equals_a_tile_by_tile_dispatch(lib):
    rng = random.Random(1)
    for k in range(60):
        runs = copy([Run(rng.randint(1, 300), rng.randint(1, 90), rng.choice([1, 3, 4, 16, 64]), True)
                     for _ in range(rng.randint(1, 5))])
        places = rng.choice([1, 7, 64, 2048])
        assert lib.finish(runs, len(runs), places) == dispatched(runs, places), k


def test_choice_is_never_later_than_the_plans_blocks(lib):
    """300 launches: where the choice changes the blocks the launch ends earlier, and none has more
    tiles than allowed or blocks of more than 64."""
    rng = random.Random(2)
    changed, gain = 0, []
    for k in range(300):
        own = launch(rng)
        new = copy(own)
        lib.choose(new, len(new), PLACES, (1 << 31) - 1, True)
        assert all(1 <= r.tpb <= 64 and (r.segs, r.members) == (o.segs, o.members) for r, o in zip(new, own))
        if [r.tpb for r in new] == [r.tpb for r in own]:
            continue
        changed += 1
        a, b = dispatched(own), dispatched(new)
        assert b < a, (k, [(r.segs, r.members, r.tpb) for r in own], [r.tpb for r in new], a, b)
        gain.append(a / b)
    assert changed > 50 and max(gain) > 1.1


def test_fixed_blocks_and_the_tile_limit_are_kept(lib):
    runs = copy([Run(1061 + 20 * i, 16, 4, i != 2) for i in range(8)])  # widths of 201 templates, 2^20 bins
    lib.choose(runs, 8, PLACES, (1 << 31) - 1, True)
    assert runs[2].tpb == 4 and all(runs[i].tpb > 4 for i in range(8) if i != 2)
    runs = copy([Run(1110, 238, 64, True)])
    lib.choose(runs, 1, PLACES, 1110 * 4, True)  # no more tiles than the plan's blocks
    assert runs[0].tpb >= 60


@pytest.mark.parametrize("whole", [False, True])
def test_choice_costs_the_caller_little(lib, whole):
    """Every search and batch call pays for the choice: under 10 us for eight jobs on the hosts it was
    written on; ten times that is refused (instrumented hosts are not timed)."""
    if "asan" in os.environ.get("LD_PRELOAD", ""):
        pytest.skip("address sanitizer preloaded")
    rng = random.Random(3)
    most = 0.0
    for _ in range(40):
        own = launch(rng)
        best = 1.0
        for _ in range(20):
            new = copy(own)
            t = time.perf_counter()
            lib.choose(new, len(new), PLACES, (1 << 31) - 1, whole)
            best = min(best, time.perf_counter() - t)
        most = max(most, best)
    assert most < 100e-6, most


def as_runs(items):
    """A batch as the library gives it: few jobs each by itself, of many those of all spectra but the
    last together per width group."""
    jobs = [r for item in items for r in item]
    if len(jobs) <= 16 or (len(jobs) <= 32 and sum(r.segs * -(-r.members // r.tpb) for r in jobs) >= 2 * PLACES):
        return copy(jobs)
    per = len(items[0])
    head = [Run(sum(i[g].segs for i in items[:-1]), items[0][g].members, items[0][g].tpb, True) for g in range(per)]
    return copy(head + list(items[-1]))


def test_choice_for_batches(lib):
    """Batches of 2 to 150 uneven spectra: where the blocks change, the launch, whose tiles come
    spectrum by spectrum, ends earlier."""
    rng = random.Random(5)
    changed, gain = 0, []
    for k in range(150):
        one = launch(rng)
        items = []
        for _ in range(int(2 ** rng.uniform(1, 7.2))):
            share = rng.uniform(0.25, 1.0)
            items.append([Run(max(1, int(r.segs * share)), r.members, r.tpb, True) for r in one])
        runs = as_runs(items)
        before = [r.tpb for r in runs]
        per = len(one)
        lib.choose(runs, len(runs), PLACES, (1 << 31) - 1, len(runs) == per * len(items))
        new = [r.tpb for r in runs][-per:]
        assert [r.tpb for r in runs] == new * (len(runs) // per)
        if [r.tpb for r in runs] == before:
            continue
        changed += 1
        own = copy([r for item in items for r in item])
        got = copy([Run(r.segs, r.members, t, True) for item in items for r, t in zip(item, new)])
        a, b = lib.finish(own, len(own), PLACES), lib.finish(got, len(got), PLACES)  # every tile in order
        assert b < a, (k, len(items), [(r.segs, r.members, r.tpb) for r in one], new, a, b)
        gain.append(a / b)
    assert changed > 30 and max(gain) > 1.1


def test_candidate_passes_with_many_hits_keep_their_blocks(lib):
    """A candidate pass reads a tile's hits back one after the other: blocks grow only where a larger
    tile expects few."""
    assert lib.allowed(60, 16, 928, 11.7) and lib.allowed(64, 4, 993, 9.0)
    for pre in (-1.0, 0.0, 2.0, 5.4, 6.0):
        assert not lib.allowed(28, 16, 928, pre) and not lib.allowed(9, 4, 928, pre)
        assert lib.allowed(16, 16, 928, pre) and lib.allowed(8, 16, 928, pre)
