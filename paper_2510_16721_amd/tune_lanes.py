"""Autotuner of the LJ force kernel's lanes per atom (1, 2, 4 .. 32 lanes of
a wavefront share one atom's candidates).

For LJ FCC vacancy-hop bands over a range of sizes (atoms x moving images), each lane
count is timed on the band stepped alone (HIP-event phase timing of the force
stage, cfneb_step_profiled) and, where many such bands fit, on a full batch of them
(whole steps).  A band keeps its count alone and in a batch, so a batch never changes
its sums; the count therefore has to do for both: the fewest lanes within MARGIN of the
fastest alone, among those that cost a full batch at most BATCH_MARGIN, and no more lanes
than a smaller band.  A relaxation (one moving image, made and stepped by one call) is
never in a batch: the fewest lanes within 3 % of the fastest.  Both for FP32 and for FP64
bands, whose pairs cost more.  The picks become the rows of csrc/lj_lanes_table.h, which the library compiles in and looks up at creation.

    python -m paper_2510_16721_amd.tune_lanes            # measure and print
    python -m paper_2510_16721_amd.tune_lanes --write    # and rewrite the table
(then rebuild the library).
"""
import argparse
import math
import os
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
TABLE = os.path.join(HERE, "csrc", "lj_lanes_table.h")
LANES = (1, 2, 4, 8, 16, 32)
BAND_LANES = (1, 2, 4, 8)
MARGIN = 0.15
# What a full batch may lose to the best count there.  More lanes leave more of them idle (93
# candidates are 24 fours: three rounds of 8 lanes, two of 16) and repeat an item's work more often:
# 128 bands of 499 atoms x 5 moving images take 149, 150, 163, 179, 222 and 275 us a step with
# 1, 2, 4, 8, 16 and 32 lanes, one of them alone 70, 65, 62, 60.5, 59 and 59.
BATCH_MARGIN = {4: 0.25, 8: 0.17}
BATCH = 128
# (FCC cells per edge, images): 31 .. 97,555 atoms, 155 .. 2.1M atoms x moving images
CASES = [(2, 7), (4, 3), (3, 7), (4, 5), (4, 7), (5, 5), (8, 3), (5, 7), (10, 3), (6, 7), (8, 7), (8, 11), (11, 7),
         (14, 7), (16, 7), (16, 11), (22, 7), (29, 7), (29, 24)]
# FCC cells per edge of the relaxations: 255 .. 97,555 atoms
RELAX_CASES = [4, 6, 8, 9, 10, 11, 12, 13, 14, 16, 20, 24, 29]


def _band(n, images, fp64):
    sys.path.insert(0, os.path.dirname(HERE))
    import workloads as W
    from . import cfneb
    w = W.fcc_vacancy_hop(n, n, n, 1.5496)
    p = cfneb.default_params(cfneb.CFNEB_LJ, n_images=images, max_images=images, climb_after=-1,
                             force_fp64=fp64)
    return cfneb.Band(p, w["pos_init"], w["cell_init"], w["pos_final"], w["cell_final"]), w["n"]


def time_case(n, images, fp64=0, lanes=LANES, steps=20, warmup=5):
    """Force-stage ms per step for each lane count."""
    out = {}
    for k in lanes:
        os.environ["CFNEB_LJ_LANES"] = str(k)
        try:
            band, atoms = _band(n, images, fp64)
            band.step(warmup)
            _, _, _, ph = band.step_profiled(steps)
            out[k] = ph["force0"] / steps
            band.close()
        finally:
            del os.environ["CFNEB_LJ_LANES"]
    return atoms, out


def time_batch(n, images, count, fp64=0, steps=32):
    """ms per step of a batch of `count` such bands for each lane count."""
    sys.path.insert(0, os.path.dirname(HERE))
    import torch
    import workloads as W
    from . import cfneb
    w = W.fcc_vacancy_hop(n, n, n, 1.5496)
    p = cfneb.default_params(cfneb.CFNEB_LJ, n_images=images, max_images=images, climb_after=-1, force_fp64=fp64)
    out = {}
    for k in BAND_LANES:
        os.environ["CFNEB_LJ_LANES"] = str(k)
        try:
            batch = cfneb.Batch(count)
            for q in range(count):
                slot = batch.add(p, w["pos_init"], w["cell_init"], w["pos_final"], w["cell_final"])
                batch.bands[slot].displace_interior(W.interior_noise(q, images, w["n"]))
            batch.step(steps)  # past the first list rebuilds
            times = []
            for _ in range(3):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                batch.step(steps)
                times.append(time.perf_counter() - t0)
            out[k] = 1000 * min(times) / steps
            batch.close()
        finally:
            del os.environ["CFNEB_LJ_LANES"]
    return out


def allowed(t, batch):
    """The times alone of the counts that a full batch bears (batch None: not measured) and that
    are within MARGIN of the fastest of all, else of the fastest that it bears."""
    if batch is None:
        return dict(t)
    limit = min(batch.values())
    ok = {k: v for k, v in t.items() if batch[k] <= limit * (1.0 + BATCH_MARGIN.get(k, 1.0))}
    best = min(t.values())
    near = {k: v for k, v in ok.items() if v <= best * (1.0 + MARGIN)}
    fastest = min(ok, key=ok.get)
    return near or {fastest: ok[fastest]}


def pick(t, margin=0.03):
    """The fewest lanes within `margin` of the fastest time (ties and timing noise keep
    the simpler shape)."""
    best = min(t.values())
    return min(k for k in t if t[k] <= best * (1.0 + margin))


def table_rows(results, margin=MARGIN):
    """results: [(atom_images, {lanes: ms})] -> [(max_atom_images, lanes)], thresholds at
    the geometric mean of neighbouring sizes whose picked counts differ; a larger size never
    takes more lanes than a smaller one."""
    pts = sorted((w, pick(t, margin)) for w, t in results)
    pts = [(w, min(k for _, k in pts[:i + 1])) for i, (w, _) in enumerate(pts)]
    rows = []
    for i, (w, k) in enumerate(pts):
        if i + 1 < len(pts) and pts[i + 1][1] == k:
            continue
        if i + 1 < len(pts):
            rows.append((int(math.sqrt(w * pts[i + 1][0])), k))
        else:
            rows.append((None, k))
    return rows


def write_table(measured, path=TABLE):
    """measured: {fp64: (results, batches, relaxations)}."""
    def times(t):
        return "  ".join(f"{k}: {1000 * t[k]:8.1f}" for k in LANES if k in t)

    lines = ["// LJ lanes per atom by band size (atoms x moving images at creation): the fewest lanes",
             f"// within {100 * MARGIN:.0f} % of the fastest alone, among those that cost a full batch of such bands at",
             f"// most {100 * BATCH_MARGIN[4]:.0f} % (4 lanes) or {100 * BATCH_MARGIN[8]:.0f} % (8), and no more than a smaller band takes.  Relaxations",
             "// (one moving image, never in a batch) by atoms: the fewest lanes within 3 % of the fastest,",
             "// and no more than a smaller one takes.  Written by tune_lanes.py from vacancy-hop bands:",
             "// force-stage times alone, and whole steps of the batch (us per step; "
             f"{BATCH} bands, fewer",
             "// from 19,500 atom-images on)."]
    for fp64, (results, batches, relax) in measured.items():
        lines.append(f"// FP{64 if fp64 else 32} bands, atom-images:")
        for w, t in sorted(results):
            lines.append(f"//   {w:>9d}           " + times(t))
            if w in batches:
                lines.append("//             in a batch " + times(batches[w]))
        lines.append(f"// FP{64 if fp64 else 32} relaxations, atoms:")
        for w, t in sorted(relax):
            lines.append(f"//   {w:>9d}           " + times(t))
    lines += ["#ifndef CFNEB_LJ_LANES_TABLE_H", "#define CFNEB_LJ_LANES_TABLE_H", "",
              "struct LjLanesEntry {", "    long long max_atom_images;", "    int lanes;", "};"]
    for fp64, (results, batches, relax) in measured.items():
        rows = table_rows([(w, allowed(t, batches.get(w))) for w, t in results])
        last, tail = ("9223372036854775807LL", "LL") if not fp64 else ("2147483647", "")
        lines.append(f"static const LjLanesEntry kLjLanes{'Fp64' if fp64 else 'Table'}[] = {{")
        lines += [f"    {{{last if w is None else str(w) + tail}, {k}}}," for w, k in rows]
        lines += ["};", f"static const LjLanesEntry kLjLanesRelax{'Fp64' if fp64 else ''}[] = {{"]
        lines += [f"    {{{2147483647 if w is None else w}, {k}}}," for w, k in table_rows(relax, 0.03)]
        lines.append("};")
    lines += ["", "#endif", ""]
    with open(path, "w") as f:
        f.write("\n".join(lines))


def main(argv=None):
    ap = argparse.ArgumentParser()
    ap.add_argument("--write", action="store_true", help="rewrite csrc/lj_lanes_table.h")
    ap.add_argument("--out", default=TABLE, help="where --write puts the table")
    args = ap.parse_args(argv)
    import torch
    if not torch.cuda.is_available():
        raise SystemExit("tune_lanes: needs a HIP device")

    def say(what, t):
        print(f"tune_lanes: {what}: " + "  ".join(f"K={k} {1000 * t[k]:.1f} us" for k in t), flush=True)

    measured = {}
    for fp64 in (0, 1):
        name, results, batches, relax = f"FP{64 if fp64 else 32}", [], {}, []
        for n, images in CASES:
            atoms, t = time_case(n, images, fp64, BAND_LANES)
            work = atoms * (images - 2)
            say(f"{name} {atoms} atoms x {images - 2} moving images", t)
            results.append((work, t))
            count = min(BATCH, int(2.5e6 / work))
            if count >= 16:
                batches[work] = time_batch(n, images, count, fp64)
                say(f"a batch of {count}", batches[work])
        for n in RELAX_CASES:
            atoms, t = time_case(n, 3, fp64)
            say(f"{name} {atoms} atoms x 1 moving image", t)
            relax.append((atoms, t))
        measured[fp64] = (results, batches, relax)
        print("tune_lanes: table", table_rows([(w, allowed(t, batches.get(w))) for w, t in results]),
              "relaxations", table_rows(relax, 0.03), flush=True)
    if args.write:
        write_table(measured, args.out)
        print(f"tune_lanes: wrote {args.out}", flush=True)


if __name__ == "__main__":
    main()
