"""Autotuner for the library's launch parameters.

For one model and workload it sweeps each tunable (see minsr_set_tunable)
over its candidate values, times the phase the tunable governs with the
library's HIP-event phase timers over a few steps that do not update the
parameters, keeps the fastest value, and records the choice in a JSON cache
keyed by device architecture, shape bucket and precision.  `apply` reads the
cache and sets the recorded values on a model; batches are built from models
tuned this way.

A sample_r other than 0 takes the matrix-core recurrence away from every
evaluation of the model too, at any number of samples.  It is therefore timed
with an evaluation of the same samples, and 0 stays unless another value is
faster by more than timings of the same kernels differ.

    tunable      phase timed                  candidates
    gram_split   Gram tiles + reduction       0 (heuristic), 1, 2, 4, 8, 16, 32
    eloc_grid    local-energy recurrence      0 (one per item), 256, 512, 1024, 2048
    sample_r     sampling + an evaluation     0 (built-in), 1, 4 (vector forms; no effect on the
                                              sampling of FP32 chains of 64 or 128 units)
    jac_parts    Jacobian reverse pass        0 (built-in), 1, 2, 4 (the per-sample kernel)
"""
import json
import os

import torch

from . import F64, FORM_BF16_FP64, FORM_FP64_REF

CANDIDATES = {
    "gram_split": (0, 1, 2, 4, 8, 16, 32),
    "eloc_grid": (0, 256, 512, 1024, 2048),
    "sample_r": (0, 1, 4),
    "jac_parts": (0, 1, 2, 4),
}
PHASES = {
    "gram_split": ("gram", "gram_reduce"),
    "eloc_grid": ("eloc",),
    "sample_r": ("sample",),
    "jac_parts": ("jacobian",),
}
# sample_r: the least of some rounds over the values in turn, and the share of
# the built-in choice's time below which another value is kept (one
# kernel against itself: up to 7 % apart at 39 us, 3 % at 49, 1.5 % at 155)
SAMPLE_R_ROUNDS = 3
SAMPLE_R_GAIN = 0.9
# version of the tunables' meaning, part of a cache entry's key; entries
# without one date from when sample_r 1 was the built-in choice (0 was not
# recorded) and jac_parts and the FP64 Gram's split belonged to other kernels
KEY_VERSION = 2
DEFAULT_CACHE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "autotune_cache.json")


def _unversioned_key(model, Ns, form):
    arch = torch.cuda.get_device_properties(model.device).gcnArchName.split(":")[0]
    d = model.desc
    return "%s/dim%d/H%d/N%d/Ns%d/cplx%d/form%d" % (arch, d.dim, d.hidden, model.N, Ns,
                                                   int(d.complex_head), form)


def shape_key(model, Ns, form):
    return "%s/%s/v%d" % (_unversioned_key(model, Ns, form),
                          "f64" if model.desc.compute_dtype == F64 else "f32", KEY_VERSION)


def _time_phase(model, ham, Ns, form, phases, reps):
    mom = torch.zeros(model.Np, dtype=torch.float64, device=model.device)
    outs = model.step_outputs(Ns)
    kw = dict(form=form, apply_update=False, outputs=outs)
    model.step(ham, Ns, 0.01, 1e-3, 0.0, mom, 1, 0, **kw)       # warm caches and code
    torch.cuda.synchronize()
    model.timing_begin(reps)
    for i in range(reps):
        model.step(ham, Ns, 0.01, 1e-3, 0.0, mom, 1, i, **kw)
    torch.cuda.synchronize()
    ms, n = model.timing_read()
    return sum(ms[p] for p in phases) / max(n, 1)


def _time_evaluation(model, Ns, reps):
    """ms of one evaluation of Ns samples"""
    sigma = model.sample(Ns, key=1, counter=0)[0]
    model.logpsi(sigma)
    start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    start.record()
    for _ in range(reps):
        model.logpsi(sigma)
    end.record()
    torch.cuda.synchronize()
    return start.elapsed_time(end) / reps


def tune(model, ham, Ns, form=FORM_BF16_FP64, reps=5, keys=None, cache=DEFAULT_CACHE):
    """Sweep the tunables one at a time (in the order of CANDIDATES), set the
    best value of each on the model, and record the result in the cache.
    Returns {key: (best_value, {value: ms})}; of sample_r the built-in choice
    and the values clearly faster than it."""
    result = {}
    for key in keys or CANDIDATES:
        times = {}
        for _ in range(SAMPLE_R_ROUNDS if key == "sample_r" else 1):
            for v in CANDIDATES[key]:
                model.set_tunable(key, v)
                t = _time_phase(model, ham, Ns, form, PHASES[key], reps)
                if key == "sample_r":
                    t += _time_evaluation(model, Ns, reps)
                times[v] = min(t, times.get(v, t))
        if key == "sample_r":
            times = {v: t for v, t in times.items() if v == 0 or t < SAMPLE_R_GAIN * times[0]}
        best = min(times, key=times.get)
        model.set_tunable(key, best)
        result[key] = (best, times)
    if cache:
        data = load(cache)
        data[shape_key(model, Ns, form)] = {k: v[0] for k, v in result.items()}
        tmp = cache + ".tmp"
        with open(tmp, "w") as f:
            json.dump(data, f, indent=1, sort_keys=True)
        os.replace(tmp, cache)
    return result


def load(cache=DEFAULT_CACHE):
    if not os.path.exists(cache):
        return {}
    with open(cache) as f:
        return json.load(f)


def apply(model, Ns, form=FORM_BF16_FP64, cache=DEFAULT_CACHE):
    """Set the cached launch parameters for this model's shape bucket;
    returns the applied dict (empty if the bucket was never tuned)."""
    data = load(cache)
    entry = data.get(shape_key(model, Ns, form))
    if entry is None:   # of an unversioned entry, what still means the same
        old = data.get(_unversioned_key(model, Ns, form), {})
        keep = ("eloc_grid",) if form == FORM_FP64_REF else ("eloc_grid", "gram_split")
        entry = {k: old[k] for k in keep if k in old}
    for k, v in entry.items():
        model.set_tunable(k, v)
    return entry
