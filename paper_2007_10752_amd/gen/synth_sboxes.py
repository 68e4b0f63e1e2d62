"""Search for the S-box gate networks and store them in sbox_networks.txt.

Builds sbox_synth.cpp with g++, runs it once per S-box and restriction
(restarts split over worker processes with distinct seeds) and keeps, per
box, the network that makes the round cheapest: gates plus the second-use
XORs that remain after second_use_plan folds masks into gates.  A
restriction (--restrict, bit masks of S-box inputs) asks the search for
networks whose gates can take those inputs' key masks (SBOX_RESTRICT in
sbox_synth.cpp); the inputs that matter are the shared ones, 0, 1, 4 and 5.
Run by hand when the search changes; the committed sbox_networks.txt is what
the emitter reads, so a normal build does not search.

    python -m paper_2007_10752_amd.gen.synth_sboxes --restarts 2000 --jobs 8
    python -m paper_2007_10752_amd.gen.synth_sboxes --restarts 1400 --restrict 1,2,16,32

With --walk SECONDS it shrinks networks by local search instead
(sbox_walk.cpp): each job starts from the stored network or, every other
one, from a fresh result of sbox_synth.cpp.  With --keys N it searches over
the S-box inputs and the key masks of N of its second uses together, so that a
mask's XOR counts like a gate and is saved where the mask fits into one.

    python -m paper_2007_10752_amd.gen.synth_sboxes --walk 300 --jobs 8
    python -m paper_2007_10752_amd.gen.synth_sboxes --walk 300 --jobs 8 --keys 1
"""
import argparse
import concurrent.futures as cf
import itertools
import os
import subprocess
import tempfile

from .des_tables import SBOX
from .networks import (NETWORKS_PATH, SECOND_USES, foldable, format_networks, live_signals,
                       load_networks, lut3, parse_network, second_use_plan, verify_network)

HERE = os.path.dirname(os.path.abspath(__file__))


def _build(tmpdir, name="sbox_synth", keys=0):
    exe = os.path.join(tmpdir, "%s%d" % (name, keys))
    subprocess.run(["g++", "-O2", "-DKEYS=%d" % keys, "-o", exe, os.path.join(HERE, name + ".cpp")],
                   check=True)
    return exe


def _without_keys(text):
    """A network over the S-box inputs and key masks (signals from 6 on), as
    sbox_walk.cpp prints it, with the masks 0: gates that then pass a signal on
    are left out.  foldable() says which masks fit back in."""
    gates, outs, of = [], [None] * 4, {q: q for q in range(6)}
    for line in text.splitlines():
        f = line.split()
        if f and f[0] == "g":
            v, ops, imm = int(f[1]), [int(x) for x in f[2:5]], int(f[5])
            sig = [of.get(x, 0) for x in ops]  # (a mask's slot: any signal, ignored)
            new = 0
            for idx in range(8):
                val = [(idx >> (2 - i)) & 1 if ops[i] in of else 0 for i in range(3)]
                new |= lut3(imm, *val) << idx
            live = live_signals((*sig, new))
            same = len(live) == 1 and all(
                lut3(new, *(b if x in live else 0 for x in sig)) == b for b in (0, 1))
            if same:
                of[v] = live.pop()
            else:
                of[v] = 6 + len(gates)
                gates.append((*sig, new))
        elif f and f[0] == "out":
            outs[int(f[1])] = (of[int(f[2])], int(f[3]))
    return {"gates": gates, "outs": outs}


def _walk(exe, box, seconds, seed, start, keys=()):
    vals = [str(v) for row in SBOX[box] for v in row]
    r = subprocess.run([exe, str(seconds), str(seed), "0.6", "4"] + vals + [str(q) for q in keys],
                       check=True, input=format_networks({box: start}), capture_output=True, text=True)
    return _without_keys(r.stdout)


def _run(exe, box, restarts, seed, restrict, lookahead):
    vals = [str(v) for row in SBOX[box] for v in row]
    env = dict(os.environ, SBOX_RESTRICT=str(restrict), SBOX_LOOKAHEAD=str(lookahead))
    r = subprocess.run([exe, str(restarts), str(seed)] + vals, check=True,
                       capture_output=True, text=True, env=env)
    lines = r.stdout.splitlines()
    if not lines or int(lines[0].split()[1]) >= 1 << 20:
        return None  # every restart of this job was dropped
    return parse_network(r.stdout)


def round_cost(nets):
    """Gates plus second-use XORs per round for a full set of networks."""
    _, folded = second_use_plan(nets)
    return sum(len(n["gates"]) for n in nets.values()) + 16 - len(folded)


def _fold_sets(net):
    return frozenset(frozenset(c) for n in range(5) for c in itertools.combinations((0, 1, 4, 5), n)
                     if foldable(net, c))


def choose(cands):
    """Per box, the candidate networks; returns the combination of least
    round_cost (candidates dominated within their box, more gates and no fold
    set the other lacks, are dropped first)."""
    pruned = {}
    for box, nets in cands.items():
        keep = []
        for n in sorted(nets, key=lambda n: len(n["gates"])):
            fs = _fold_sets(n)
            if any(len(k["gates"]) <= len(n["gates"]) and fs <= _fold_sets(k) for k in keep):
                continue
            keep.append(n)
        pruned[box] = keep
    boxes = sorted(pruned)
    best, best_cost = None, None
    for combo in itertools.product(*(pruned[b] for b in boxes)):
        nets = dict(zip(boxes, combo))
        cost = round_cost(nets)
        if best_cost is None or cost < best_cost:
            best, best_cost = nets, cost
    return best


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--restarts", type=int, default=1000)
    ap.add_argument("--jobs", type=int, default=os.cpu_count() or 4)
    ap.add_argument("--seed", type=int, default=1)
    ap.add_argument("--boxes", default="0,1,2,3,4,5,6,7")
    ap.add_argument("--restrict", default="0",
                    help="comma-separated bit masks of restricted inputs, one search each")
    ap.add_argument("--lookahead", type=int, default=int(os.environ.get("SBOX_LOOKAHEAD", "0")))
    ap.add_argument("--walk", type=float, default=0, help="seconds of local search per job")
    ap.add_argument("--keys", type=int, default=0, help="second uses whose key masks join the walk")
    args = ap.parse_args()
    boxes = [int(b) for b in args.boxes.split(",")]
    masks = [int(m) for m in args.restrict.split(",")]
    try:
        current = load_networks()
    except FileNotFoundError:
        current = {}
    cands = {b: [current[b]] for b in range(8) if b in current}
    if args.walk:
        with tempfile.TemporaryDirectory() as td, cf.ThreadPoolExecutor(args.jobs) as pool:
            synth = _build(td)
            walk = [_build(td, "sbox_walk", k) for k in range(args.keys + 1)]

            def job(box, j):
                seed = args.seed * 1000003 + box * 7919 + j
                start = current.get(box) if j % 2 == 0 else None
                sets = list(itertools.combinations([e % 6 for e in SECOND_USES if e // 6 == box], args.keys))
                keys = sets[j // 2 % len(sets)] if sets else ()
                return _walk(walk[len(keys)], box, args.walk, seed,
                             start or _run(synth, box, 1, seed, 0, 0), keys)
            futs = {pool.submit(job, b, j): b for j in range(args.jobs) for b in boxes}
            for fut in cf.as_completed(futs):
                verify_network(futs[fut], fut.result())
                cands.setdefault(futs[fut], []).append(fut.result())
        return _store(choose(cands))
    with tempfile.TemporaryDirectory() as td:
        exe = _build(td)
        per_job = max(1, args.restarts // args.jobs)
        with cf.ThreadPoolExecutor(args.jobs) as pool:
            futs = {}
            for box in boxes:
                for mask in masks:
                    for j in range(args.jobs):
                        seed = args.seed * 1000003 + box * 7919 + mask * 104729 + j
                        futs[pool.submit(_run, exe, box, per_job, seed, mask, args.lookahead)] = (box, mask)
            found = {}
            for fut in cf.as_completed(futs):
                box, mask = futs[fut]
                net = fut.result()
                if net is None:
                    continue
                verify_network(box, net)
                key = (box, mask)
                if key not in found or len(net["gates"]) < len(found[key]["gates"]):
                    found[key] = net
    for (box, mask), net in sorted(found.items()):
        print("S%d restrict %d: %d gates" % (box + 1, mask, len(net["gates"])))
        cands.setdefault(box, []).append(net)
    _store(choose(cands))


def _store(best):
    _, folded = second_use_plan(best)
    for box in sorted(best):
        print("S%d: %d gates" % (box + 1, len(best[box]["gates"])))
    print("round: %d gates + %d XORs (%d second-use masks folded)"
          % (sum(len(n["gates"]) for n in best.values()), 48 - len(folded), len(folded)))
    with open(NETWORKS_PATH, "w") as f:
        f.write(format_networks(best))


if __name__ == "__main__":
    main()
