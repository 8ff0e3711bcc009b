"""Host rules of the attention launch's shared tiles (csrc/split_plan.h),
compiled on their own: no GPU."""
import random
import subprocess

import pytest

from paper_2607_01817_amd import build

DRIVER = r"""
#include <cstdio>
#include "split_plan.h"
using namespace hcms;
constexpr int64_t kSlot = 68 * 1024;
// region mem r n_cu            -> part ml count (offsets), slots counters n_cu
// plan W nkb n_cu mem r tail   -> n_whole n_split halves ways has_scratch
// copies W nkb n_cu mem r bytes -> n_whole n_split halves ways ride idle, two copies of these bytes
// use stream role capturing    -> region wait record, a launch of one pool
int main() {
    char what[16];
    SplitPool pool;
    while (std::scanf("%15s", what) == 1) {
        long long W, mem, tail;
        int nkb, n_cu, r;
        if (what[0] == 'r') {
            if (std::scanf("%lld %d %d", &mem, &r, &n_cu) != 3) return 1;
            const SplitScratch s = split_region(reinterpret_cast<void *>(mem), r, n_cu, kSlot);
            std::printf("%lld %lld %lld %d %d %d\n", (long long)s.part - mem, (long long)s.ml - mem,
                        (long long)s.count - mem, s.slots, s.counters, s.n_cu);
        } else if (what[0] == 'c') {
            if (std::scanf("%lld %d %d %lld %d %lld", &W, &nkb, &n_cu, &mem, &r, &tail) != 6) return 1;
            const SplitScratch s = split_region(reinterpret_cast<void *>(mem), r, n_cu, kSlot);
            const RidingSplit p = plan_riding(W, nkb, n_cu, &s, static_cast<double>(tail), 2);
            std::printf("%d %d %d %d %d %lld\n", p.split.n_whole, p.split.n_split, p.split.halves, p.split.ways,
                        p.ride, (long long)idle_cus(p.split, n_cu));
        } else if (what[0] == 'u') {
            int role, capturing;
            if (std::scanf("%lld %d %d", &mem, &role, &capturing) != 3) return 1;
            const void *stream = reinterpret_cast<void *>(mem);
            bool wait = false, record = false;
            const int at = pool.find(stream, role, capturing, &wait);
            if (at >= 0) {
                pool.own(at, stream);
                record = pool.records(at, capturing);
                if (record) pool.recorded(at);
            }
            std::printf("%d %d %d\n", at, wait, record);
        } else {
            if (std::scanf("%lld %d %d %lld %d %lld", &W, &nkb, &n_cu, &mem, &r, &tail) != 6) return 1;
            SplitScratch s = split_region(mem < 0 ? nullptr : reinterpret_cast<void *>(mem), r, n_cu, kSlot);
            s.tail = tail;
            const TailSplit p = plan_split(W, nkb, n_cu, mem < 0 ? nullptr : &s);
            std::printf("%d %d %d %d %d\n", p.n_whole, p.n_split, p.halves, p.ways, p.part && p.ml && p.count);
        }
    }
    std::printf("%lld %lld\n", (long long)split_bytes(256, kSlot), (long long)split_counter_bytes(256));
}
"""
MEM = 1 << 40      # an address that nothing reads
SLOT = 68 * 1024


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined",
                    "-fno-sanitize-recover=undefined", "-I", build.CSRC, str(d / "driver.cpp"),
                    "-o", str(d / "driver")], check=True)

    def ask(lines):
        r = subprocess.run([str(d / "driver")], input="\n".join(lines) + "\n", text=True,
                           capture_output=True)
        assert r.returncode == 0, (r.returncode, r.stderr[-500:])
        return [tuple(map(int, ln.split())) for ln in r.stdout.splitlines()]

    return ask


def test_regions_fill_the_scratch_without_overlap(rules):
    *regions, (total, counters) = rules([f"region {MEM} {r} 256" for r in range(3)])
    spans = []
    for part, ml, count, slots, n_count, n_cu in regions:
        assert n_cu == 256 and slots == n_count
        spans += [(part, slots * (SLOT - 4096)), (ml, slots * 4096), (count, n_count * 4)]
        assert part % 16 == 0 and ml % 16 == 0 and count % 4 == 0
        assert count >= total - counters    # the zeroed end
    end = 0
    for at, n in sorted(spans):
        assert at == end
        end = at + n
    assert end == total < 64 << 20


@pytest.mark.parametrize("mem", [0, -1])
def test_launches_without_scratch_split_no_tile_by_segments(rules, mem):
    """A context whose scratch could not be had (an empty region), and a call
    without one: whole tiles or halves, whatever the size."""
    if mem == 0:
        part, ml, count, slots, n_count, n_cu = rules(["region 0 0 256"])[0]
        assert (slots, n_count, n_cu) == (0, 0, 256)
    asked = [(W, nkb, n) for n in (1, 2, 3, 80, 256) for W in (1, 2, 40, 100, 128, 129, 155, 256, 1100)
             for nkb in (1, 12, 900)]
    got = rules([f"plan {W} {nkb} {n} {mem} 0 -1" for W, nkb, n in asked])
    for (W, nkb, n), (whole, split, halves, ways, scratch) in zip(asked, got):
        t = W % n
        assert whole + split == W and ways == 1 and scratch == 0
        assert (split, halves) == ((t, 2) if n >= 2 and 0 < 2 * t <= n else (0, 1))


def test_an_unset_scratch_splits_nothing(rules):
    """Zero compute units in the scratch (a region that was never filled in)."""
    assert rules([f"plan {W} 900 0 0 0 -1" for W in (1, 155, 1100)])[:3] == \
        [(W, 0, 1, 1, 0) for W in (1, 155, 1100)]


@pytest.mark.parametrize("r", [0, 1, 2])
def test_split_units_fit_the_scratch(rules, r):
    slots = (512, 256, 192)[r]
    asked = [(W, nkb, tail) for W in range(1, 520) for nkb in (11, 12) for tail in (-1, 0, 40, 76, 170)]
    got = rules([f"plan {W} {nkb} 256 {MEM} {r} {tail}" for W, nkb, tail in asked])
    for (W, nkb, tail), (whole, split, halves, ways, scratch) in zip(asked, got):
        assert whole + split == W and halves in (1, 2) and ways in (1, 3)
        assert split in (0, min(W % 256 if tail < 0 else tail, W))
        assert scratch == (ways == 3) and (ways == 1 or (nkb >= 12 and split * halves * ways <= slots))


def test_two_rounds_of_segments_only_where_they_are_shorter(rules):
    """More than half a round of tiles: segments over two rounds from 40 key
    blocks on, from 64 with more than 160 of 256 tiles, and not beyond 170."""
    asked = [(t, nkb) for t in (129, 160, 161, 170, 171) for nkb in (12, 39, 40, 63, 64, 900)]
    got = rules([f"plan {256 + t} {nkb} 256 {MEM} 0 -1" for t, nkb in asked])
    for (t, nkb), (whole, split, halves, ways, _) in zip(asked, got):
        shared = t <= 170 and nkb >= (40 if t <= 160 else 64)
        assert (whole, split, halves, ways) == ((256, t, 1, 3) if shared else (256 + t, 0, 1, 1)), (t, nkb)
    # Not where two launches share the rounds.
    asked = [(t, r) for t in (129, 160, 170) for r in (0, 1)]
    assert rules([f"plan 256 900 256 {MEM} {r} {t}" for t, r in asked])[:len(asked)] == [(256, 0, 1, 1, 0)] * 6


@pytest.mark.parametrize("W,nkb,mb,want", [
    (440, 878, 100, (440, 0, 1, 1, 1)),      # 72 CUs idle over a long whole round
    (156, 50, 29, (156, 0, 1, 1, 1)),        # whole tiles leave 100 CUs, segments over two rounds 44
    (411, 1644, 100, (256, 155, 1, 3, 1)),   # long keys: two rounds, and time for the copies in the second
    (296, 32, 20, (256, 40, 1, 3, 1)),       # thirds leave 136 CUs, sixths 16
    (296, 32, 77, (256, 40, 2, 1, 1)),       # more copies than 136 CUs move meanwhile: halves leave 176
    (296, 1184, 100, (256, 40, 2, 3, 0)),    # long keys: sixths, the copies behind them
    (250, 878, 10, (250, 0, 1, 1, 0)),       # 6 CUs idle
    (384, 16, 200, (256, 128, 2, 1, 0)),     # more copies than the idle CUs can move meanwhile
    (512, 878, 100, (512, 0, 1, 1, 0)),      # none idle
    # The middle launches of RIDING_FORMS in the GPU tests, three chunks of one head.
    (36, 141, 9, (0, 36, 2, 3, 1)), (63, 250, 16, (0, 63, 1, 3, 1)), (98, 391, 26, (0, 98, 2, 1, 1)),
    (145, 579, 38, (0, 145, 1, 3, 1)), (184, 735, 48, (184, 0, 1, 1, 1)),
])
def test_split_of_a_launch_with_copies(rules, W, nkb, mb, want):
    """Worked by hand from the rates beside plan_riding."""
    assert rules([f"copies {W} {nkb} 256 {MEM} 0 {mb * 10 ** 6}"])[0][:5] == want


@pytest.mark.parametrize("mem", [0, MEM])
def test_copies_ride_beside_at_least_an_eighth_of_the_units(rules, mem):
    asked = [(W, nkb, mb) for W in range(1, 520, 3) for nkb in (8, 20, 60, 900) for mb in (1, 30, 400)]
    got = rules([f"copies {W} {nkb} 256 {mem} 0 {mb * 10 ** 6}" for W, nkb, mb in asked])
    plain = rules([f"plan {W} {nkb} 256 {mem} 0 -1" for W, nkb, mb in asked])
    assert any(g[4] for g in got[:len(asked)])
    for (W, nkb, mb), (whole, split, halves, ways, ride, idle), p in zip(asked, got, plain):
        assert whole + split == W and (mem or ways == 1)
        assert idle >= 32 if ride else (whole, split, halves, ways) == p[:4]
        assert ways == 1 or (nkb >= 12 and split * halves * ways <= 512)


def _uses(rules, uses):
    return rules([f"use {stream} {role} {capturing}" for stream, role, capturing in uses])[:len(uses)]


def test_one_main_and_one_compute_stream_record_no_event(rules):
    got = _uses(rules, [(7, 0, 0), (8, 1, 0)] * 3)
    assert got == [(0, 0, 0), (1, 0, 0)] * 3


def test_a_capture_on_another_stream_keeps_a_region_of_its_own(rules):
    """Warmed up on stream 7, captured on stream 9, then used on 7 again and on
    11: 9's region is never handed on, and no capture waits for an event."""
    got = _uses(rules, [(7, 0, 0), (9, 0, 1), (7, 0, 0), (11, 0, 0), (12, 0, 1)])
    assert got == [(0, 0, 0), (2, 0, 0), (0, 0, 1), (0, 1, 1), (-1, 0, 0)]


@pytest.mark.parametrize("seed", range(20))
def test_a_region_changes_streams_only_behind_an_event(rules, seed):
    """Random streams, roles and captures: where a region's launch follows one
    of another stream, it waits for an event recorded behind that launch, and
    neither of the two is in a capture."""
    rng = random.Random(seed)
    streams = [0] + rng.sample(range(1, 100), rng.randint(1, 5))
    uses = [(rng.choice(streams), rng.randint(0, 1), int(seed % 2 and rng.random() < 0.1))
            for _ in range(200)]
    last, handed = {}, 0
    for (stream, role, capturing), (r, wait, record) in zip(uses, _uses(rules, uses)):
        if r < 0:
            continue
        if r in last and last[r][0] != stream:
            handed += 1
            assert wait and last[r][1] and not capturing and not last[r][2]
        else:
            assert not wait
        captured = capturing or (r in last and last[r][0] == stream and last[r][2])
        assert not (record and capturing)
        last[r] = (stream, record, captured)
    assert handed > 0 or seed % 2 or len(streams) <= 3
