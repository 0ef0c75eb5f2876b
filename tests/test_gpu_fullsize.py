"""Full-size steps in the configuration ``bench.py`` times (GPU).

Below a ReLU or a max pool a gradient depends on choices between values that may almost
tie.  Rounding decides such a choice and one of them moves a single element by up to its own
size: noise of 1e-7 on the float64 oracle's convolution outputs moves an element of
``s3b2.c.conv.W``'s gradient (ResNet-50, batch 16) by more than twice what the float32 oracle's
error allows, or not at all, depending on the noise's seed.  So gradients are compared under the
device's own choices, and the choices themselves with float64's up to ties of rounding size
(``gpu_util.check_decisions``).

What remains ill-conditioned in fp32 is BatchNorm over few rows.  The bar is therefore derived
from the arithmetic: for every parameter gradient, updated parameter and momentum buffer, the
device's relative L2 error against float64 must be at most 1.5 times the float32 oracle's own
under the same choices, and its largest element error (relative to the largest element) at most 3
times the float32 oracle's (neither ever has to be smaller than 1e-4; see
``gpu_util.within_fp32_error``).  The loss, a well-conditioned forward quantity, must match
float64 within 1e-5.

The out-of-core step must equal the in-core step bit for bit in the exact
bench configuration (budget, window, chunk size).
"""

import numpy as np
import pytest

import bench
from paper_2010_14109_amd import netdef, synth
from tests.gpu_util import check_under_own_choices, run_net

pytestmark = pytest.mark.gpu


def derived_check(spec, x, labels, params, loss, outs, chunk):
    e64, worst = check_under_own_choices(spec, x, labels, params, outs, chunk)
    assert abs(loss - e64["loss"][-1]) <= 1e-5 * abs(e64["loss"][-1])
    print(f"{spec['name']}: worst error / bound: relative L2 {worst[0]:.2f}, largest element "
          f"{worst[1]:.2f}", flush=True)


def bench_config(name, **over):
    spec = synth.workload(name, **over)
    net = netdef.Net(spec)
    chunk, plan = bench.choose_chunk(net, synth.budget_fraction(name), bench.window_fraction(name))
    return spec, chunk, plan


def test_plain_cnn_batch128_bench_config():
    spec, chunk, plan = bench_config("cnn")
    x, labels = synth.make_inputs(spec, 0)
    params = synth.make_params(spec, 1)
    print(f"cnn b128: budget {plan['budget']} chunk {chunk}", flush=True)
    loss, outs, st = run_net(spec, x, labels, params, budget=plan["budget"],
                             window=plan["window"], chunk=chunk)
    assert st["pool_bytes"] <= plan["budget"]
    loss0, outs0, _ = run_net(spec, x, labels, params, chunk=chunk)
    assert np.float32(loss).tobytes() == np.float32(loss0).tobytes()
    for n in outs0:
        assert outs[n].tobytes() == outs0[n].tobytes(), n
    print("cnn b128: bit-identical to in-core; checking against the oracle", flush=True)
    derived_check(spec, x, labels, params, loss, outs, chunk)


@pytest.mark.parametrize("batch,hw", [(16, 64), (4, 224)])
def test_resnet50_against_oracle(batch, hw):
    spec = synth.resnet(batch=batch, hw=hw)
    x, labels = synth.make_inputs(spec, 0)
    params = synth.make_params(spec, 1)
    net = netdef.Net(spec, keep_grads=True)
    chunk, plan = bench.choose_chunk(net, 1 / 7.5, bench.DEFAULT_WINDOW_FRAC)
    print(f"resnet50 b{batch} {hw}x{hw}: budget {plan['budget']} chunk {chunk}", flush=True)
    loss, outs, st = run_net(spec, x, labels, params, budget=plan["budget"],
                             window=plan["window"], chunk=chunk)
    assert st["pool_bytes"] <= plan["budget"]
    derived_check(spec, x, labels, params, loss, outs, chunk)


@pytest.mark.parametrize("spec", [
    synth.mlp(batch=131, width=515, depth=5, classes=67),
    synth.plain_cnn(batch=24, channels=36, depth=5, hw=23),
    synth.resnet(batch=6, hw=99, width=24, blocks=(1, 1, 1, 1)),
    synth.densenet(batch=9, hw=32, growth=8, blocks=(4, 4, 4, 4)),
    synth.unet(batch=2, hw=56, base=20, depth=3)], ids=lambda s: s["name"])
def test_networks_of_every_kind_under_own_choices(spec):
    """Every network with ReLUs at a ragged middle size, in core: gradients to rounding instead of
    to the size of a flipped choice."""
    x, labels = synth.make_inputs(spec, 0)
    params = synth.make_params(spec, 1)
    loss, outs, _ = run_net(spec, x, labels, params)
    derived_check(spec, x, labels, params, loss, outs, 2 << 20)


def test_resnet50_batch256_bench_config_matches_incore():
    spec, chunk, plan = bench_config("resnet50_b256")
    x, labels = synth.make_inputs(spec, 0)
    params = synth.make_params(spec, 1)
    print(f"resnet50 b256: budget {plan['budget']} chunk {chunk}", flush=True)
    loss, outs, st = run_net(spec, x, labels, params, budget=plan["budget"],
                             window=plan["window"], chunk=chunk, keep_grads=False)
    assert st["pool_bytes"] <= plan["budget"] and st["device_bytes_delta"] <= plan["budget"]
    loss0, outs0, _ = run_net(spec, x, labels, params, chunk=chunk, keep_grads=False)
    assert np.isfinite(loss) and np.float32(loss).tobytes() == np.float32(loss0).tobytes()
    for n in outs0:
        assert outs[n].tobytes() == outs0[n].tobytes(), n
