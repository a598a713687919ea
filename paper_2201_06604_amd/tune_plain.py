"""Tune the automatic launch shapes of mrg_generate on this GPU.

    python -m paper_2201_06604_amd.tune_plain            # time and print the table
    python -m paper_2201_06604_amd.tune_plain --write    # also rewrite csrc/mrg_tuned.h

csrc/mrg_tuned.h holds, per output kind and size class, an entry for each half of
the class and for rows that start on 4 KB pages, on 128-byte lines and anywhere:
streams per lane, threads per block, the waves a grid aims at (plan_generate chooses
the chunk count near it by the grid that comes out most evenly), the shortest chunk,
lockstep rows and XCD block order.  For each entry this script creates its
representative workloads (SIZES x COUNTS: stream counts of every kind, not powers of
two alone, streams created on the device from a fixed seed), works out the launch
shape each candidate resolves to under the automatic plan's rules (`resolve`, the
same steps plan_generate takes), times every distinct shape with mrg_generate_ex
(HIP events around launches queued behind a sleeping kernel, so that what counts is
the device's time; two passes, the second over the better shapes only) and keeps the
candidate whose times, each over the best of its workload, have the smallest mean and
largest value.  Blocks of one wave are not among the candidates: timed after their
own kind they come out evenly, but after another kernel their waves share SIMDs (2^30
fp32 uniforms of 262,144 streams 660 us after themselves, 910 after another shape).
The library must be rebuilt after --write.  Results never depend on the shapes, only
times do.
"""
import argparse
import os
import re
import sys

import numpy as np

PKG = os.path.dirname(os.path.abspath(__file__))
HEADER = os.path.join(PKG, "csrc", "mrg_tuned.h")

UNIFORM, NORMAL, EXPONENTIAL, RAW = 0, 1, 2, 3
F64, F32, U32 = 0, 1, 2
KINDS = [("uniform f64", UNIFORM, F64), ("uniform f32", UNIFORM, F32), ("raw u32", RAW, U32),
         ("normal f64", NORMAL, F64), ("normal f32", NORMAL, F32), ("exponential f64", EXPONENTIAL, F64),
         ("exponential f32", EXPONENTIAL, F32)]
CLASSES = [(256, 256), (1024, 1024), (16384, 1024), (65536, 4096), (262144, 4096)]  # streams x draws
# a class's second half starts at this many draws
HALF = [1 << 15, 1 << 20, 23_726_566, 189_812_531, 1 << 31]  # 2^24.5 and 2^27.5 among them
FIELDS = ("spl", "block", "waves", "min_units", "lock", "xcd")
# draws of each class's halves, and the stream counts timed at them (those of at least
# eight draws each): counts whose rows start on lines, powers of two among others, and
# counts whose rows do not
SIZES = [[(10_000, 1 << 16), (1 << 16, 180_000)], [(1 << 19, 900_000), (1 << 21, 3_500_000)],
         [(8_000_000, 1 << 24), (1 << 25, 48_000_000)], [(80_000_000, 1 << 27), (1 << 28, 450_000_000)],
         [(600_000_000, 1 << 30), ()]]
COUNTS = [(1024, 2048, 5120, 10240, 16384, 30720, 65536, 99328, 131072, 262144, 299008),
          (64, 640, 1600, 4992, 9984, 20032, 30016, 50048, 100032, 131136, 200000, 299968),
          (77, 555, 1001, 2252, 10007, 30011, 70001, 100003, 131077, 200003, 262143)]


def workloads(c, h, al):
    """(streams, draws) that an entry is timed on."""
    return [(S, n // S * S + (S // 3 if al == 2 else 0)) for n in SIZES[c][h] for S in COUNTS[al] if n >= 8 * S]


def read_table(path=HEADER):
    """The entries of csrc/mrg_tuned.h as [kind][class] dicts: a shape for
    each half of the class ("halves") and row alignment (pages, lines, ragged)."""
    src = open(path).read()
    body = src[src.index("kTuned[kTunedKinds][kTunedClasses][2][3] = {"):]
    nums = [tuple(int(v) for v in m.split(",")) for m in re.findall(r"\{(\s*\d+(?:\s*,\s*\d+){5})\s*\}", body)]
    assert len(nums) == len(KINDS) * len(CLASSES) * 6, len(nums)
    shapes = iter(dict(zip(FIELDS, v)) for v in nums)
    return [[{"class": c, "halves": [[next(shapes) for _ in range(3)] for _ in range(2)]}
             for c in range(len(CLASSES))] for _ in KINDS]


def write_table(table, notes, path=HEADER):
    src = open(path).read()
    cut = src.find("// Timings")
    head = src[:cut if cut >= 0 else src.index("// clang-format off")]
    tail = src[src.index("// clang-format on"):]
    one = lambda e: "{" + ", ".join(str(e[f]) for f in FIELDS) + "}"  # noqa: E731
    rows = []
    for k, (name, _, _) in enumerate(KINDS):
        rows.append(f"    {{  // {name}")
        for c in range(len(CLASSES)):
            halves = ", ".join("{" + ", ".join(one(e) for e in half) + "}" for half in table[k][c]["halves"])
            rows.append(f"        {{{halves}}},")
        rows.append("    },")
    body = ("// clang-format off\n"
            "constexpr TunedShape kTuned[kTunedKinds][kTunedClasses][2][3] = {\n" + "\n".join(rows) + "\n};\n")
    note = "".join(f"// {ln}\n" for ln in notes)
    with open(path, "w") as f:
        f.write(head + note + body + tail)


# the cost of a grid on its busiest CU, as in plan_generate
UNIT_SLOTS = (16, 16, 15, 73, 60, 32, 29)
START_SLOTS, SLOT_US, FINALIZE_US = 256, 1.0 / 2100.0, 4.0
ONE_WAVE, LOCK_FROM, GAP_WAVES, NARROW_WAVES, NARROW_FROM = 1024, 1536, 32768, 8192, 1 << 26


def alignment(S, esz):
    """0, 1, 2: rows on 4 KB pages, on 128-byte lines, anywhere."""
    return 2 if S * esz % 128 else 1 if S * esz % 4096 else 0


def kind_of(dist, dtype):
    return [(d, t) for _, d, t in KINDS].index((dist, dtype))


def grid_cost(n_sblk, units, chunks, wpb, lock, kind, spl):
    """(cost, chunk, chunks) of a grid."""
    chunk = -(-units // chunks)
    k = -(-units // chunk)
    column = not lock and 1 < k <= wpb
    blocks = n_sblk if column else -(-n_sblk // wpb) * k
    waves = -(-blocks // 256) * (k if column else wpb)
    cost = max(4 if spl > 1 else 8, waves) * (float(chunk) * UNIT_SLOTS[kind] + START_SLOTS) * spl * SLOT_US
    return cost + (FINALIZE_US if k > 1 and not column else 0.0), chunk, k


def choose_chunks(n_sblk, units, aim, most, wpb, lock, shared, least, kind, spl):
    """(chunk, waves per block) of the grid that costs least around the aim."""
    cost, chunk, _ = grid_cost(n_sblk, units, aim, wpb, lock, kind, spl)
    best = cost, chunk, wpb
    w = wpb
    while w >= 1:
        whole = w >= n_sblk
        if w < wpb and (w < least if whole else shared or w < 4):
            break
        row = -(-n_sblk // w)
        handicap = 1.01 if w == wpb else 1.04
        if row <= 256:
            r = aim * row // 256
            ks = [256 * m // row for m in range(max(1, r - r // 3), min(r + r // 2 + (1 if shared else 3), r + 7) + 1)]
        else:
            ks = range(aim - aim // 3, aim + aim // 2 + (2 if shared else 6) + 1)
        for k in ([aim] if w < wpb else []) + list(ks):
            if 1 <= k <= most:
                cost, chunk, _ = grid_cost(n_sblk, units, k, w, lock, kind, spl)
                far = float(k) / float(aim)
                cost *= handicap + 0.15 * (far - 1.0 if far > 1.0 else 1.0 / far - 1.0)
                if cost < best[0]:
                    best = cost, chunk, w
        w //= 2
    return best[1], best[2]


def resolve(entry, S, n, dist, dtype):
    """The launch shape plan_generate gives an automatic call with this table
    entry (output aligned to 256 bytes): the keys of mrg_launch_cfg."""
    esz = 8 if dtype == F64 else 4
    if "halves" in entry:
        c, entry = entry["class"], entry["halves"][1 if n >= HALF[entry["class"]] else 0]
        at = alignment(S, esz)
        one = entry[0]
        if at == 0 and c >= 3 and one["waves"] == ONE_WAVE and not one["lock"]:
            if ONE_WAVE * 64 * one["spl"] % S or ONE_WAVE * 64 * one["spl"] // S == 2:
                at = 1
        entry = entry[at]
    spl = entry["spl"]
    while spl * esz > 16:
        spl //= 2
    while spl > 1 and S % spl:
        spl //= 2
    while spl > 1 and 64 * spl > S:
        spl //= 2
    q, r = divmod(n, S)
    cnt_max = q + (1 if r else 0)
    units_max = (cnt_max + 1) // 2 if dist == NORMAL else cnt_max
    n_sblk = -(-S // (64 * spl))
    most = max(1, -(-units_max // entry["min_units"]))
    shared = entry["lock"] and S * esz % 128 != 0
    wide = entry["block"] // 64
    aim = entry["waves"]
    if shared and 5 * n_sblk < 4 * (-(-n_sblk // wide) * wide):
        aim = max(aim, GAP_WAVES)
    if not entry["lock"] and n_sblk < 4 and q * S >= NARROW_FROM:
        aim = max(aim, NARROW_WAVES)
    w = max(1, min(most, -(-aim // n_sblk)))
    block, chunk = entry["block"], max(1, -(-units_max // w))
    chosen = n_sblk * w > ONE_WAVE
    if chosen:
        least = 4 if dist == NORMAL and q * S < NARROW_FROM else 1
        chunk, wpb = choose_chunks(n_sblk, units_max, w, most, wide, entry["lock"], shared, least,
                                   kind_of(dist, dtype), spl)
        block = 64 * wpb
    nch = -(-units_max // chunk) if units_max else 0
    if nch > 65535:
        chunk = -(-units_max // 65535)
        nch = -(-units_max // chunk)
    lock = 1 if entry["lock"] and n_sblk * nch >= LOCK_FROM and (shared or n_sblk * 64 >= block) else 0
    xcd = entry["xcd"]
    wpb = block // 64
    column = not lock and 1 < nch <= wpb
    if not chosen and not lock and not column and n_sblk * nch < 2048 and block > 256:
        block, wpb = 256, 4
    if not lock and (n_sblk if column else -(-n_sblk // wpb) * nch) % 8:
        xcd = 0
    return {"block": block, "chunk": chunk, "nontemporal": 1 if (S * esz) % 128 == 0 else 0,
            "arith": 2, "streams_per_lane": spl, "xcd_remap": xcd, "lockstep": lock}


def candidates(dist, dtype, c, al):
    plain = dist in (UNIFORM, RAW)
    # full-size rows on lines: rows in step are for fp64 uniforms, whose entry is the
    # shape of the throughput case; the other kinds run free there
    locks = (0,) if c == 4 and al == 0 else (0, 1)
    for spl in (1,) if al == 2 else (1, 2, 4) if dtype != F64 and plain else (1, 2):
        for block in (256, 512, 1024):
            for waves in (512, 1024, 2048, 3072, 4096, 6144, 8192, 12288, 16384, 24576, 32768):
                for min_units in (4, 16):
                    for lock in locks:
                        for xcd in (0, 1):
                            yield dict(spl=spl, block=block, waves=waves, min_units=min_units, lock=lock, xcd=xcd)


def tune(against=(), classes=range(len(SIZES)), kinds=range(len(KINDS))):
    import ctypes

    import torch

    import paper_2201_06604_amd as P
    table = read_table()
    new = [[{"class": c, "halves": [list(h) for h in e["halves"]]} for c, e in enumerate(row)] for row in table]
    notes = []
    torch.cuda.set_device(0)
    creator = P.mrg_creator_init([1234567, 7654321, 1111111, 2222222, 3333333, 4444444])
    streams = P.mrg_streams_create_device(creator, 299968)
    room = torch.empty((1 << 30) + 299968, dtype=torch.float64, device="cuda")

    def time_of(S, n, dist, dtype, key, reps):
        cfg = dict(key)
        out = room if dtype == F64 else room.view(torch.float32 if dtype == F32 else torch.int32)
        P.mrg_generate(streams, n, dist, dtype, 1.0, out=out, cfg=cfg, n_streams=S)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        if n < 1 << 24:
            torch.cuda._sleep(40000 * reps)  # the launches queue up behind it
        a.record()
        for _ in range(reps):
            P.mrg_generate(streams, n, dist, dtype, 1.0, out=out, cfg=cfg, n_streams=S)
        b.record()
        b.synchronize()
        return a.elapsed_time(b) / reps * 1e3

    others = []  # the automatic call of other builds
    for path in against:
        lib = ctypes.CDLL(path)
        lib.mrg_generate.argtypes = P.lib().mrg_generate.argtypes
        others.append(lib.mrg_generate)

    def best_of_others(S, n, dist, dtype, reps):
        """The fastest other build, us; infinite without any."""
        best = [float("inf")]
        for call in others:
            for _ in range(4):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                call(P.MRG_GEN_MRG32K3A, streams.data_ptr(), S, n, dist, dtype, 1.0, room.data_ptr(), None)
                if n < 1 << 24:
                    torch.cuda._sleep(40000 * reps)
                a.record()
                for _ in range(reps):
                    call(P.MRG_GEN_MRG32K3A, streams.data_ptr(), S, n, dist, dtype, 1.0, room.data_ptr(), None)
                b.record()
                b.synchronize()
                best.append(a.elapsed_time(b) / reps * 1e3)
        return min(best)

    for c in classes:
        for h in range(2):
            for al in range(3):
                for k in kinds:
                    name, dist, dtype = KINDS[k]
                    work = workloads(c, h, al)
                    if not work:  # nothing larger is timed
                        new[k][c]["halves"][h][al] = dict(new[k][c]["halves"][h - 1][al])
                        continue
                    was = table[k][c]["halves"][h][al]
                    cands = [was] + list(candidates(dist, dtype, c, al))
                    if (c, dist, dtype) == (4, UNIFORM, F64) and al < 2:  # the shape of the throughput case
                        cands = [e for e in cands if (e["spl"], e["block"], e["lock"], e["xcd"]) == (2, 512, 1, 1)]
                    logs, lost, line = [], [], []
                    for S, n in work:
                        keys = [tuple(sorted(resolve(e, S, n, dist, dtype).items())) for e in cands]
                        reps = max(2, min(8, (1 << 23) // n))
                        first = {key: time_of(S, n, dist, dtype, key, reps) for key in dict.fromkeys(keys)}
                        limit = 1.12 * min(first.values())
                        again = {key: min(t, *(time_of(S, n, dist, dtype, key, reps) for _ in range(5)))
                                 for key, t in first.items() if t <= limit or key == keys[0]}
                        best = min(again.values())
                        times = np.array([again.get(key, first[key]) for key in keys])
                        other = best_of_others(S, n, dist, dtype, reps)
                        logs.append(np.log(times / best))
                        lost.append(np.maximum(0.0, np.log(times / other) - 0.02))
                        line.append((S, n, other, times))
                    logs, lost = np.array(logs), np.array(lost)
                    score = logs.mean(0) + 0.5 * logs.max(0) + 2.0 * lost.mean(0) + lost.max(0)
                    pick = int(np.argmin(score))
                    if score[0] <= score[pick] + 0.01:
                        pick = 0
                    new[k][c]["halves"][h][al] = dict(cands[pick])
                    over = f"{np.exp(logs.mean(0)[pick]):.2f} and {np.exp(logs.max(0)[pick]):.2f}"
                    notes.append(f"{name}, class {c} half {h}{(' pages', ' lines', ' ragged')[al]}: {over}")
                    print(f"{name}: " + "; ".join(f"{S} of {n} ({o:.1f}) {t[0]:.1f} -> {t[pick]:.1f}" for S, n, o, t in line),
                          over, new[k][c]["halves"][h][al], flush=True)
    return new, notes


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--write", action="store_true", help="rewrite csrc/mrg_tuned.h with the result")
    ap.add_argument("--out", default=HEADER, help="where --write puts the header (default: csrc/mrg_tuned.h)")
    ap.add_argument("--against", default="", help="other builds of the library, by commas: an entry slower than their "
                                                  "automatic shapes is marked down by what it loses")
    ap.add_argument("--classes", default="0,1,2,3,4", help="the size classes to time")
    ap.add_argument("--kinds", default="0,1,2,3,4,5,6", help="the output kinds to time")
    a = ap.parse_args()
    table, notes = tune([p for p in a.against.split(",") if p], [int(c) for c in a.classes.split(",")],
                        [int(k) for k in a.kinds.split(",")])
    if a.write:
        if a.out != HEADER:
            with open(a.out, "w") as f:
                f.write(open(HEADER).read())
        write_table(table, ["Time over the fastest candidate's, mean and most over an entry's workloads:"] + notes, path=a.out)
        print("wrote", a.out)


if __name__ == "__main__":
    sys.exit(main())
