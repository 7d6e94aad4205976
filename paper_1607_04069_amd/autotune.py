"""Launch-shape autotuner for the step kernels (one case or a batch).

Every launch shape (pm_launch_shape: particles per lane in flight, register
budget, workgroups sharing the particles, LDS deposit variant, steps between
cell sorts) computes the same particles, charges and diagnostics; only the
speed differs.  The tuner therefore times candidate shapes on the live state --
the steps it takes are real steps of the run -- and keeps the fastest, in
stages, each timed by the calls that its fields act on: push variant and
workgroup count by single steps, with a runoff of the best few re-timed in
alternation; then, by calls of several steps, a batch's lanes, the deposit
variant and the sort interval.  The workgroup counts tried are those that leave
calls of several steps their full resident wave.  Choices are cached in a JSON
file keyed by the device and a signature of the workload, so a later run of the
same workload starts from the tuned shape without timing anything.
"""
import json
import math
import os
import time

CACHE_ENV = "PICMCC_TUNE_CACHE"
# part of the key: a call of several steps takes one launch a step (shapes chosen
# when it took two are not looked up)
STEP_FORM = "one-launch"


def cache_path():
    return os.environ.get(CACHE_ENV, os.path.join(os.path.expanduser("~"), ".cache", "picmcc",
                                                  "launch_shapes.json"))


def _device():
    """Architecture and compute-unit count of device 0, e.g. gfx950/256CU."""
    import torch
    props = torch.cuda.get_device_properties(0)
    return f"{props.gcnArchName.split(':')[0]}/{props.multi_processor_count}CU"


def signature(params):
    """Workload key: precision, and per case the grid size, particles (to a
    factor of sqrt 2) and collision regime (pressure to a factor of 2)."""
    items = sorted((int(p["n_cells"]), int(round(2 * math.log2(max(p["np_e"] + p["np_i"], 1)))),
                    int(round(math.log2(max(p["p_pa"], 1e-3))))) for p in params)
    fp64 = int(bool(params[0].get("fp64", 0)))
    return f"fp64={fp64};cases={len(items)};" + ",".join(f"{a}/{b}/{c}" for a, b, c in items)


# Shapes tuned on an MI355X and shipped with the package; the user cache (written
# by tune) takes precedence.
SHIPPED = os.path.join(os.path.dirname(os.path.abspath(__file__)), "launch_shapes.json")


def _read(path):
    try:
        with open(path) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def _load():
    data = _read(SHIPPED)
    data.update(_read(cache_path()))
    return data


def _store(key, shape, rate):
    path = cache_path()
    data = _read(path)
    data[key] = {"shape": shape, "particle_steps_per_s": rate}
    os.makedirs(os.path.dirname(path), exist_ok=True)
    tmp = path + ".tmp"
    with open(tmp, "w") as f:
        json.dump(data, f, indent=1, sort_keys=True)
    os.replace(tmp, path)


class _Target:
    """A Case or a Batch seen through one interface."""

    def __init__(self, obj):
        self.obj = obj
        self.cases = obj.cases if hasattr(obj, "cases") else [obj]

    def particle_steps(self):
        return sum(c.sample_diagnostics()["particle_steps"] for c in self.cases)

    def rate(self, steps, single=False):
        """Particle-steps/s of a call of several steps, or of as many calls of one."""
        import torch
        torch.cuda.synchronize()
        p0 = self.particle_steps()
        t0 = time.perf_counter()
        if single:
            for _ in range(steps):
                self.obj.step(1)
        else:
            self.obj.step(steps)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        return (self.particle_steps() - p0) / dt


def workload_key(obj, params):
    return "|".join((_device(), "batch" if hasattr(obj, "cases") else "case", STEP_FORM, signature(params)))


def tune(obj, params, steps=None, use_cache=True, log=None):
    """Tune the launch shape of a Case or Batch (params: the parameter dicts of
    its cases) and leave the best shape set.  Returns (shape, particle-steps/s,
    source) with source "cache" or "timed"."""
    key = workload_key(obj, params)
    if use_cache:
        hit = _load().get(key)
        if hit:
            obj.set_launch_shape(**hit["shape"])
            return obj.launch_shape(), hit["particle_steps_per_s"], "cache"
    t = _Target(obj)
    base = obj.launch_shape()
    obj.set_launch_shape(work_groups=0)
    resident = obj.launch_shape()["work_groups"]
    is_batch = hasattr(obj, "cases")
    mults = (1, 2, 3) if is_batch else (0.5, 1)
    sort0 = base["sort_interval"] or 25
    if steps is None:
        steps = 200 if is_batch else 100
    steps = sort0 * max(1, -(-steps // sort0))     # whole sort intervals per trial

    def trial(single, **kw):
        obj.set_launch_shape(**kw)
        obj.step(4)                                  # settle caches after the change
        r = max(t.rate(steps, single), t.rate(steps, single))   # the better of two, against transients
        if log:
            log(f"  shape {kw}{', single steps' if single else ''}: {r:.3e} particle-steps/s")
        return obj.launch_shape(), r

    def runoff(tried, single, k=3, rounds=2):
        """Re-time the k best distinct shapes so far in alternation: the state
        evolves during the search, so trials taken at different times are not
        quite comparable; alternating shapes sees the same state for each."""
        uniq = []
        for sh, r in sorted(tried, key=lambda e: -e[1]):
            if sh not in [u for u, _ in uniq]:
                uniq.append((sh, r))
            if len(uniq) == k:
                break
        score = {i: [] for i in range(len(uniq))}
        for _ in range(rounds):
            for i, (sh, _) in enumerate(uniq):
                obj.set_launch_shape(**sh)
                obj.step(4)
                score[i].append(t.rate(steps, single))
        i_best = max(score, key=lambda i: sum(score[i]) / len(score[i]))
        if log:
            for i, (sh, _) in enumerate(uniq):
                log(f"  runoff {sh}: {sum(score[i]) / len(score[i]):.3e} particle-steps/s")
        return uniq[i_best][0]

    # stage 1: push variant and workgroups of single steps, each trial over whole
    # sort intervals so all see the same mix
    shape = dict(runoff([trial(True, unroll=unroll, waves=waves, work_groups=max(1, int(resident * m)), deposit_mode=1,
                               sort_interval=sort0, lanes=1)
                         for unroll in (8, 16) for waves in (0, 6) for m in mults], True))
    if is_batch:
        # stage 1b: lanes stepped concurrently
        shape = dict(runoff([trial(False, **dict(shape, lanes=lanes)) for lanes in (1, 2, 3, 4)], False))
    # stage 2: deposit variant
    shape = dict(max((trial(False, **dict(shape, deposit_mode=dm)) for dm in (1, 0)), key=lambda e: e[1])[0])
    # stage 3: sort interval, timed over several intervals
    best = None
    long_steps = 200 if is_batch else 100
    for k in sorted({10, 20, 25, 50, 100}):
        obj.set_launch_shape(**dict(shape, sort_interval=k))
        obj.step(k)
        r = max(t.rate(long_steps), t.rate(long_steps))
        if log:
            log(f"  sort_interval {k}: {r:.3e} particle-steps/s")
        if best is None or r > best[1]:
            best = (obj.launch_shape(), r)
    shape = dict(best[0])
    obj.set_launch_shape(**shape)
    shape = obj.launch_shape()
    _store(key, shape, best[1])
    return shape, best[1], "timed"
