"""Tuner for the persistent step kernel: for every grid side present in a
population, times each compiled (workgroup size, exchange variant)
configuration on the live population and keeps the fastest; then times, on the
whole population, a few launch schedules of the size groups (which stream each
side's launch goes to, in which order; several grid sides only) together with
the number of steps per launch (the whole call, or the call split into shorter
launches).  Results are cached in a JSON file keyed by
(device name, side, population bucket, whether every robot has a CU, spring
model, the library's configuration list for that side)."""
import hashlib
import json
import os
import time

import torch

from . import api

CUS = 256  # compute units of an MI355X


def _bucket(count):
    b = 1
    while b < count:
        b *= 2
    return b


def _sub_population(pop, n):
    """The robots of side n of a built population, rebuilt alone from the same
    per-voxel inputs and physics, so one side can be timed in isolation."""
    cls, w = pop.query()
    idx = [r for r, m in enumerate(pop.sides) if m == n]
    offs = [0]
    for m in pop.sides:
        offs.append(offs[-1] + m ** 3)
    sel = torch.cat([torch.arange(offs[r], offs[r + 1], device=cls.device) for r in idx])
    sub = api.Population([n] * len(idx), params=pop.params, stream=pop.stream)
    sub.build_from_voxels(cls[sel].contiguous(), w[sel].contiguous())
    return sub


def _time(p, steps, reps=2):
    """Best of `reps` timed calls of `steps` steps, after one untimed call of the
    same length (which captures that call's step graph)."""
    p.reset()
    p.step(steps)
    best = float("inf")
    for _ in range(reps):
        p.reset()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        p.step(steps)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    return best


def tune(pop, steps=200, cache_path=None, verbose=False):
    """Tunes `pop` in place (it must be built); returns {side: (block, variant, seconds)}
    and leaves the chosen steps per launch (0: the whole call) in pop.steps_per_launch.
    With several grid sides each side is timed on a copy of its own robots, since
    a step of the whole population runs every side.  The population is reset to
    its build state afterwards."""
    dev_name = torch.cuda.get_device_name(pop.device)
    cache = {}
    if cache_path and os.path.exists(cache_path):
        cache = json.load(open(cache_path))
    counts = {}
    for n in pop.sides:
        counts[n] = counts.get(n, 0) + 1
    result = {}
    for n, cnt in sorted(counts.items()):
        configs = api.persist_configs(n)
        lib = hashlib.sha256(repr(configs).encode()).hexdigest()[:12]
        # the library's default depends on whether every robot of the population
        # has a CU; one side's robots alone may have one where the whole do not
        default = pop.persist_variant(n)
        key = "%s|n=%d|R<=%d%s%s|%s" % (dev_name, n, _bucket(cnt), "|alone" if len(pop.sides) <= CUS else "",
                                        "|dash" if pop.dashpots else "", lib)
        if key in cache:
            b, v, t = cache[key]
            try:
                pop.set_persist_variant(n, b, v)
                result[n] = (b, v, t)
                continue
            except api.SoftRobotError:
                pass  # not usable for this population (e.g. spring parameters set directly): time again
        target = pop if len(counts) == 1 else _sub_population(pop, n)
        times = []
        for b, v in configs:
            if bool(v & 16) != pop.dashpots:
                continue  # kernels for the other spring model
            try:
                target.set_persist_variant(n, b, v)
            except api.SoftRobotError:
                continue  # e.g. voxel-rebuilt parameters after pop_set_spring_params
            dt = _time(target, steps)
            if verbose:
                print("side %d block %d variant %d: %.4f s" % (n, b, v, dt), flush=True)
            times.append((b, v, dt))
        # keep the default unless another configuration is clearly (3 %) faster,
        # so that timing noise does not flip between equivalent kernels
        best = min(times, key=lambda q: q[2])
        for q in times:
            if (q[0], q[1]) == default and q[2] <= 1.03 * best[2]:
                best = q
        if target is not pop:
            target.close()
        pop.set_persist_variant(n, best[0], best[1])
        result[n] = best
        cache[key] = list(best)
    # launch schedule and steps per launch, together, on the whole population
    # with the configurations above, timed on calls of at least 2000 steps so
    # that the launch count is representative.  Schedules (several sides
    # only): each side's launch on a stream of its own, largest first (the
    # default), or the sides dealt largest first round-robin over 2..4
    # streams, or over three streams back and forth.  Steps per launch: the
    # whole call, or launches of 1000 or 250 steps (sides sharing a stream
    # then take turns).  The default pair is kept unless another is 3 % faster.
    desc = sorted(counts, reverse=True)
    scheds = [list(range(len(desc)))]
    if len(counts) > 1:
        scheds += [[i % k for i in range(len(desc))] for k in (2, 3, 4)]
        scheds.append([(i // 3 % 2) * (2 - i % 3) + (1 - i // 3 % 2) * (i % 3) for i in range(len(desc))])
    skey = "%s|launch|%s|%s" % (dev_name, ",".join("%d:%d" % (n, c) for n, c in sorted(counts.items())),
                                ",".join("%d:%d:%d" % (n, r[0], r[1]) for n, r in sorted(result.items())))
    if skey in cache:
        lanes, spl = list(cache[skey][0]), int(cache[skey][1])
    else:
        length = max(steps, 2000)
        times = []
        for lanes in scheds:
            if len(counts) > 1:
                pop.set_schedule(desc, lanes)
            for c in (0, 1000, 250):
                if c >= length:
                    continue
                pop.set_step_config(api._lib.SR_STEP_AUTO, 0, c)
                t = _time(pop, length)
                if verbose:
                    print("schedule %s, steps per launch %s: %.4f s" % (lanes, c or "all", t), flush=True)
                times.append((lanes, c, t))
        best = min(times, key=lambda q: q[2])
        chosen = times[0] if times[0][2] <= 1.03 * best[2] else best
        lanes, spl = chosen[0], chosen[1]
        cache[skey] = [lanes, spl]
    if len(counts) > 1:
        pop.set_schedule(desc, lanes)
    pop.set_step_config(api._lib.SR_STEP_AUTO, 0, spl)
    pop.steps_per_launch = spl
    pop.reset()
    if cache_path:
        tmp = cache_path + ".tmp"
        json.dump(cache, open(tmp, "w"), indent=1)
        os.replace(tmp, cache_path)
    return result
