"""Tune the automatic launch shapes of mrg_generate on this GPU.

    python -m paper_2201_06604_amd.tune_plain            # time and print the table
    python -m paper_2201_06604_amd.tune_plain --write    # also rewrite csrc/mrg_tuned.h

csrc/mrg_tuned.h holds, per output kind and size class, an entry for each half of
the class and for rows that start on 128-byte lines and rows that do not: streams
per lane, threads per block, the waves a grid aims at (which sets the chunk of
draws per work-item), the shortest chunk, lockstep rows and XCD block order.  For
each entry this script creates its representative workloads (WORKLOADS: streams
and draws per stream, streams created on the device from a fixed seed), works out
the launch shape each candidate resolves to under the automatic plan's rules
(`resolve`, the same steps plan_generate takes), times every distinct shape with
mrg_generate_ex (HIP events around launches queued behind a sleeping kernel, so
that what counts is the device's time; two passes, the second over the better
shapes only) and keeps the candidate whose times, each over the best of its
workload, have the smallest geometric mean.  The library must be rebuilt after
--write.  Results never depend on the shapes, only times do.
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
# per class and half: workloads whose rows start on lines, and workloads whose rows do not
WORKLOADS = [
    [([(64, 156), (256, 64), (1024, 16)], [(100, 157), (1001, 20), (7, 2000)]),
     ([(256, 256), (64, 2048), (2048, 64)], [(333, 300), (1001, 150)])],
    [([(1024, 512), (64, 8192), (8192, 64)], [(1001, 500), (100, 5000)]),
     ([(1024, 1024), (256, 8192), (16384, 128)], [(1001, 2000), (10007, 200)])],
    [([(16384, 1024), (4096, 2048), (1024, 8192)], [(10007, 1000), (1001, 8000)]),
     ([(10240, 4883), (65536, 512), (1024, 40000)], [(10007, 4997), (100003, 400)])],
    [([(65536, 2048), (16384, 8192), (1024, 100000)], [(100003, 1000), (10007, 10000)]),
     ([(65536, 4096), (262144, 1024), (4096, 65536)], [(100003, 3000), (10007, 30000)])],
    [([(262144, 4096), (65536, 16384), (16384, 60000)], [(100003, 5369), (262143, 4096), (10007, 80000)]), None],
]


def read_table(path=HEADER):
    """The entries of csrc/mrg_tuned.h as [kind][class] dicts: a shape for
    each half of the class ("halves") and row alignment (aligned, ragged)."""
    src = open(path).read()
    body = src[src.index("kTuned[kTunedKinds][kTunedClasses][2][2] = {"):]
    nums = [tuple(int(v) for v in m.split(",")) for m in re.findall(r"\{(\s*\d+(?:\s*,\s*\d+){5})\s*\}", body)]
    assert len(nums) == len(KINDS) * len(CLASSES) * 4, len(nums)
    shapes = iter(dict(zip(FIELDS, v)) for v in nums)
    return [[{"class": c, "halves": [[next(shapes) for _ in range(2)] for _ in range(2)]}
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
            "constexpr TunedShape kTuned[kTunedKinds][kTunedClasses][2][2] = {\n" + "\n".join(rows) + "\n};\n")
    note = "".join(f"// {ln}\n" for ln in notes)
    with open(path, "w") as f:
        f.write(head + note + body + tail)


def resolve(entry, S, n, dist, dtype):
    """The launch shape plan_generate gives an automatic call with this table
    entry (output aligned to 256 bytes): the keys of mrg_launch_cfg."""
    esz = 8 if dtype == F64 else 4
    if "halves" in entry:
        entry = entry["halves"][1 if n >= HALF[entry["class"]] else 0][1 if S * esz % 128 else 0]
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
    waves = entry["waves"]
    if entry["lock"] and S * esz % 128 and n_sblk < 1024:
        waves = max(waves, 32768)
    w = -(-waves // n_sblk)
    w = min(w, -(-units_max // entry["min_units"]))
    w = max(w, 1)
    chunk = max(1, -(-units_max // w))
    nch = -(-units_max // chunk) if units_max else 0
    if nch > 65535:
        chunk = -(-units_max // 65535)
        nch = -(-units_max // chunk)
    lock = 1 if entry["lock"] and n_sblk * nch >= 2048 else 0
    xcd = entry["xcd"]
    block = entry["block"]
    wpb = block // 64
    column = not lock and 1 < nch <= wpb
    if not lock and not column and n_sblk * nch < 2048 and block > 256:
        block, wpb = 256, 4
    if xcd and (n_sblk if column else -(-n_sblk // wpb) * nch) % 8:
        xcd = 0
    return {"block": block, "chunk": chunk, "nontemporal": 1 if (S * esz) % 128 == 0 else 0,
            "arith": 2, "streams_per_lane": spl, "xcd_remap": xcd, "lockstep": lock}


def candidates(dist, dtype, cls, ragged):
    plain = dist in (UNIFORM, RAW)
    spls = (1,) if ragged else (1, 2, 4) if dtype != F64 and plain else (1, 2)
    # full-size rows on lines: lockstep pays for fp64 uniforms, whose entry is
    # the shape of the throughput case; the other kinds run free there
    locks = (0,) if cls == 4 and not ragged else (0, 1)
    for spl in spls:
        for block in (128, 256, 512, 1024):
            for waves in (512, 1024, 2048, 4096, 8192, 16384, 32768):
                for min_units in (4, 16, 32, 96):
                    for lock in locks:
                        for xcd in (0, 1):
                            yield dict(spl=spl, block=block, waves=waves, min_units=min_units, lock=lock, xcd=xcd)


def tune(verbose=True):
    import torch

    import paper_2201_06604_amd as P
    table = read_table()
    new = [[{"class": c, "halves": [list(h) for h in e["halves"]]} for c, e in enumerate(row)] for row in table]
    notes = []
    torch.cuda.set_device(0)
    creator = P.mrg_creator_init([1234567, 7654321, 1111111, 2222222, 3333333, 4444444])
    streams = P.mrg_streams_create_device(creator, 262144)

    def time_of(S, n, dist, dtype, out, key, reps):
        cfg = dict(key)
        P.mrg_generate(streams, n, dist, dtype, 1.0, out=out, cfg=cfg, n_streams=S)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        if n < 1 << 24:
            torch.cuda._sleep(40000 * reps)  # the launches queue up behind it
        a.record()
        for _ in range(reps):
            P.mrg_generate(streams, n, dist, dtype, 1.0, out=out, cfg=cfg, n_streams=S)
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / reps * 1e3

    for c, halves in enumerate(WORKLOADS):
        for h, both in enumerate(halves):
            for ragged in range(2):
                for k, (name, dist, dtype) in enumerate(KINDS):
                    if both is None:  # nothing larger is timed
                        new[k][c]["halves"][h][ragged] = dict(new[k][c]["halves"][h - 1][ragged])
                        continue
                    if (c, ragged, dist, dtype) == (4, 0, UNIFORM, F64):
                        continue
                    cands = [table[k][c]["halves"][h][ragged]] + list(candidates(dist, dtype, c, ragged))
                    ratios = []
                    line = []
                    for S, per in both[ragged]:
                        n = S * per
                        out = P.new_output(n, dtype)
                        keys = [tuple(sorted(resolve(e, S, n, dist, dtype).items())) for e in cands]
                        reps = max(2, min(12, (1 << 23) // n))
                        first = {key: time_of(S, n, dist, dtype, out, key, reps) for key in dict.fromkeys(keys)}
                        limit = 1.25 * min(first.values())
                        again = {key: min(t, *(time_of(S, n, dist, dtype, out, key, 2 * reps) for _ in range(5)))
                                 for key, t in first.items() if t <= limit or key == keys[0]}
                        best = min(again.values())
                        ratios.append([again.get(key, first[key]) / best for key in keys])
                        line.append((S, per, again[keys[0]], [again.get(key, first[key]) for key in keys]))
                        del out
                    score = np.log(ratios).mean(0) + 0.5 * np.log(ratios).max(0)
                    pick = int(np.argmin(score))
                    if score[0] <= score[pick] + 0.01:
                        pick = 0
                    new[k][c]["halves"][h][ragged] = dict(cands[pick])
                    text = f"{name}: " + "; ".join(f"{S} x {per} {was:.1f} -> {now[pick]:.1f} us"
                                                    for S, per, was, now in line)
                    notes.append(text)
                    if verbose:
                        print(text, new[k][c]["halves"][h][ragged], flush=True)
    return new, notes


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--write", action="store_true", help="rewrite csrc/mrg_tuned.h with the result")
    ap.add_argument("--out", default=HEADER, help="where --write puts the header (default: csrc/mrg_tuned.h)")
    a = ap.parse_args()
    table, notes = tune()
    if a.write:
        if a.out != HEADER:
            with open(a.out, "w") as f:
                f.write(open(HEADER).read())
        write_table(table, ["Timings (MI355X, us; streams x draws: the previous table's shape -> this one's):"] + notes, path=a.out)
        print("wrote", a.out)


if __name__ == "__main__":
    sys.exit(main())
