"""Helpers of the GPU tests: run a registered network through the library."""

import numpy as np

from oracle.interp import run as oracle_run
from oracle.lower import lower
from paper_2010_14109_amd import netdef, ooc


def run_net(spec, x, labels, params, *, budget=ooc.UNLIMITED, window=None, chunk=2 << 20,
            policy="C", keep_grads=True, momentum_state=None, steps=1, inspect=None,
            wait="oldest", host_limit=None, fixed=None, layout="pool", expose=()):
    """One (or more) training steps on device 0.  Returns (loss, outputs, stats) with
    outputs = {name: array} for every PARAM, STATE and OUTPUT variable; the TEMPs named in
    ``expose`` are registered as OUTPUTs.  ``inspect(ctx, net)``, when given, runs after the
    steps."""
    net = netdef.Net(spec, keep_grads=keep_grads)
    for name in expose:
        shape, dtype, _ = net.meta[name]
        net.meta[name] = (shape, dtype, ooc.OUTPUT)
        net.var_kinds[net.var(name)] = ooc.OUTPUT
    ctx = ooc.Context(0)
    try:
        net.register(ctx)
        ctx.set_chunk(chunk)
        ctx.set_budget(budget)
        if window is not None:
            ctx.set_window(window)
        ctx.set_policy(policy)
        ctx.set_wait_order(wait)
        if host_limit is not None:
            ctx.set_host_limit(host_limit)
        if fixed is not None:
            ctx.set_fixed_distance(*fixed)
        ctx.set_layout(layout)
        ctx.build_schedule()
        ctx.prepare()
        net.view(ctx, "x")[...] = x
        net.view(ctx, "labels")[...] = labels
        for name in net.param_names():
            net.view(ctx, name)[...] = params[name]
        for name in net.names:
            if name.startswith("m:"):
                st = (momentum_state or {}).get(name)
                net.view(ctx, name)[...] = 0 if st is None else st
        ctx.upload()
        mu = spec["optimizer"]["momentum"]
        losses = [ctx.step(spec["optimizer"]["lr"], mu) for _ in range(steps)]
        if inspect is not None:
            inspect(ctx, net)
        ctx.download()
        outs = {}
        for name in net.names:
            if net.meta[name][2] in (ooc.PARAM, ooc.STATE, ooc.OUTPUT):
                outs[name] = np.array(net.view(ctx, name))
        return losses[-1], outs, ctx.stats()
    finally:
        ctx.close()


def persistent_host_bytes(spec, keep_grads=True):
    """Bytes of the pinned slots of the persistent variables (4 KiB-aligned each)."""
    net = netdef.Net(spec, keep_grads=keep_grads)
    return sum((b + 4095) // 4096 * 4096 for b, k in zip(net.var_bytes, net.var_kinds)
               if k != ooc.TEMP)


STAGING_BYTES = 2 << 30   # the staging slots a host limit reserves


def check_under_own_choices(spec, x, labels, params, outs, chunk, tol=1e-4):
    """Every gradient, updated parameter and momentum buffer of a step in ``outs`` (as run_net
    returns them, first step, gradients kept) against float64 under the device's own choices.
    They are read from a second run, in core, with the ReLU outputs and max-pool indices as
    OUTPUTs, whose results have to equal ``outs`` bit for bit.  Returns the float64 oracle's
    values and the largest ratios of error to bound (``within_fp32_error``)."""
    names = decision_vars(spec)
    _, dev, _ = run_net(spec, x, labels, params, chunk=chunk, expose=names)
    for name in outs:
        assert outs[name].tobytes() == dev[name].tobytes(), name
    reg = lower(spec, keep_grads=True)
    choices = {n: dev[n].reshape(s) for n, s in ((v["name"], v["shape"]) for v in reg["vars"])
               if n in names}
    assert len(choices) == len(names)
    e64, e32 = (oracle_run(reg, x, labels, {k: v.astype(t) for k, v in params.items()}, dtype=t,
                           decisions=choices) for t in (np.float64, np.float32))
    check_decisions(spec, dev, e64, e32)
    worst = (0.0, 0.0)
    for name, val in outs.items():
        if name != "loss":
            l2, mx = within_fp32_error(name, val, e64[name], e32[name], tol)
            worst = (max(worst[0], l2), max(worst[1], mx))
    return e64, worst


def rel_l2(a, b):
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def rel_max(a, b):
    """Largest element error relative to the largest element of b."""
    a = np.asarray(a, dtype=np.float64).reshape(-1)
    b = np.asarray(b, dtype=np.float64).reshape(-1)
    return float(np.abs(a - b).max(initial=0.0) / max(np.abs(b).max(initial=0.0), 1e-30))


def rel_err(a, b):
    """The larger of the relative L2 error and the element-wise one (rel_max): one wrong
    element among millions barely moves the norm but shows in the largest element error."""
    return max(rel_l2(a, b), rel_max(a, b))


def decision_vars(spec):
    """Variables that hold the choices of a network's forward: the ReLU outputs, whose sign is
    the backward's mask, and the max pools' index variables."""
    return ([L["name"] for L in spec["layers"] if L["op"] == "relu"] +
            [L["name"] + ".idx" for L in spec["layers"] if L["op"] == "maxpool"])


def check_decisions(spec, dev, e64, e32, tol=1e-5):
    """The device's choices are those of float64 up to ties of rounding size.  A ReLU's output
    itself has to be within the float32 oracle's error of float64 (``within_fp32_error``), which
    bounds every value whose sign the two disagree on.  The input value at a max pool's index has
    to be the window's maximum within three times the float32 oracle's largest error of that
    maximum."""
    flips = total = 0
    for L in spec["layers"]:
        name = L["name"]
        if L["op"] == "relu":
            within_fp32_error(name, dev[name], e64[name], e32[name], tol)
            flips += np.count_nonzero((np.asarray(dev[name]).reshape(e64[name].shape) > 0) !=
                                      (e64[name] > 0))
            total += e64[name].size
        elif L["op"] == "maxpool":
            idx = np.asarray(dev[name + ".idx"]).reshape(e64[name].shape).astype(np.int64)
            x, k, st, pad = e64[L["in"][0]], L["k"], L["stride"], L["pad"]
            n, p, q, c = np.indices(idx.shape, sparse=True)
            h, w = p * st + idx // k - pad, q * st + idx % k - pad
            assert idx.max() < k * k and h.min() >= 0 and w.min() >= 0, name
            assert h.max() < x.shape[1] and w.max() < x.shape[2], name
            bound = max(tol, 3 * rel_max(e32[name], e64[name])) * np.abs(e64[name]).max()
            assert np.abs(x[n, h, w, c] - e64[name]).max() <= bound, name
            flips += np.count_nonzero(idx != e64[name + ".idx"])
            total += idx.size
    print(f"{spec['name']}: {flips} of {total} choices differ from float64's", flush=True)


def within_fp32_error(name, got, ref, ref32, tol, factor=1.5, element_factor=3.0):
    """Where float32 evaluation itself is ill-conditioned (normalisation over few rows), the
    device's error against float64 is bounded by the float32 oracle's own: its relative L2 error
    at most max(tol, factor times the float32 oracle's), and its largest element error (relative
    to the largest element, an extreme value that varies more between two float32 evaluations)
    at most max(tol, element_factor times the float32 oracle's).  For gradients below a ReLU or
    a max pool both references have to be taken under the device's own choices: a choice that
    almost ties moves single elements by as much as they are large, and which ones a float32
    evaluation flips is chance, so its errors bound nothing.  Returns the two ratios error /
    bound."""
    got = np.asarray(got).reshape(np.shape(ref))
    r32 = np.asarray(ref32).reshape(np.shape(ref))
    l2 = rel_l2(got, ref) / max(tol, factor * rel_l2(r32, ref))
    mx = rel_max(got, ref) / max(tol, element_factor * rel_max(r32, ref))
    assert l2 <= 1.0 and mx <= 1.0, (name, l2, mx)
    return l2, mx
