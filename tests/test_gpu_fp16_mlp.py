"""The whole-network half-precision kernel at 16, 32 and 64 rows per workgroup, beside the launches per layer: ragged rows, one to four feature tiles per
wavefront and wavefronts without one, LayerNorm rows, narrow and wide heads; every layer's output of sampled rows against
the CPU oracle (the launch without taps must give the same actions)."""
import numpy as np
import pytest

from paper_1910_01055_amd import synth
import gpu_util as U
from test_gpu_fp16 import _check, _run_gpu

pytestmark = pytest.mark.gpu
fc = synth.fc


def _nets():
    return {
        "tiles_4_3_1": synth.small_net([fc(67, 1000, "relu"), fc(1000, 600, "relu"), fc(600, 70, "none"), fc(70, 21, "none")]),
        "ln_wide": synth.small_net([fc(30, 1000, "ln_tanh"), fc(1000, 40, "none")], head="linear"),
        "ln_odd": synth.small_net([fc(111, 257, "ln_tanh"), fc(257, 96, "relu"), fc(96, 3, "none")]),
        "wide_argmax": synth.small_net([fc(33, 130, "relu"), fc(130, 100, "none")], head="argmax"),
        "narrow_argmax": synth.small_net([fc(17, 200, "relu"), fc(200, 50, "none")], head="argmax"),
        "u8_wide_head": synth.small_net([fc(48, 130, "relu"), fc(130, 70, "none")], head="tanh", in_type="u8"),
        "aligned": synth.small_net([fc(256, 512, "relu"), fc(512, 512, "relu"), fc(512, 64, "none")]),
    }


# 16, 32 and 64 rows per workgroup at 2101, 4099 and 12005; at 16391 a second round for a few rows, or a launch per layer, which some
# take at fewer rows too
BATCHES = [1, 49, 2101, 4099, 8200, 12005, 16391]


@pytest.mark.parametrize("name", list(_nets()))
def test_the_batches_reach_every_row_count(aq, name):
    net = _nets()[name]
    P = aq.Policy(net)
    P.convert_params_fp16(*U.upload_params(synth.make_params(net)))
    plan = {batch: P.policy_fp16_plan(batch) for batch in BATCHES}
    second_round = {"narrow_argmax": 0, "u8_wide_head": 0, "aligned": 0, "ln_wide": 32}
    assert (plan[2101], plan[4099], plan[12005], plan[16391]) == (16, 32, 64, second_round.get(name, 64)), plan
    P.close()


@pytest.mark.parametrize("name", list(_nets()))
@pytest.mark.parametrize("batch", BATCHES)
def test_whole_network_half_precision_kernel(aq, name, batch):
    print(f"[fp16 mlp] {name} batch={batch}", flush=True)
    net = _nets()[name]
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    actions, outs = _run_gpu(aq, net, params, obs)
    rows = np.unique(np.minimum(np.concatenate([[0, 15, 16, 31, 32, 63, 64, batch - 2, batch - 1],
                                                np.random.default_rng(3).integers(0, batch, 24)]), batch - 1))
    rows = rows[rows >= 0]
    _check(net, params, obs[rows], actions[rows], [o.reshape(batch, -1)[rows] for o in outs], end_to_end=False)


@pytest.mark.parametrize("head", ["tanh", "argmax"])
@pytest.mark.parametrize("batch", [1, 15, 16, 17])
def test_half_precision_layers_of_few_rows(aq, head, batch):
    """A launch per layer at few rows, around the 16 rows up to which a layer takes 16 x 16 tiles: shares of K of one to
    nine k-steps, wavefronts without one, ragged features, an argmax that needs its row in one tile."""
    print(f"[fp16 few rows] {head} batch={batch}", flush=True)
    net = synth.small_net([fc(67, 2056, "relu"), fc(2056, 1104, "ln_tanh"), fc(1104, 136, "relu"), fc(136, 1032, "relu"),
                           fc(1032, 1024, "relu"), fc(1024, 37 if head == "tanh" else 18, "none")], head=head)
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    actions, outs = _run_gpu(aq, net, params, obs)
    _check(net, params, obs, actions, outs, end_to_end=False)


@pytest.mark.parametrize("hidden", [(40,), (130, 70)])
@pytest.mark.parametrize("batch", [1, 50, 4099])
def test_an_overflowing_observation_is_infinite_and_not_nan(aq, hidden, batch):
    """A binary16 overflow in front of layers without activation, all weights positive: the row's actions are +infinity
    (the features that pad a layer to whole tiles are no NaN that the next layer adds), the other rows stay finite."""
    print(f"[fp16 overflow] {hidden} batch={batch}", flush=True)
    widths = [20, *hidden]
    net = synth.small_net([fc(k, n, "none") for k, n in zip(widths, widths[1:])] + [fc(widths[-1], 6, "none")], head="linear")
    params = synth.make_params(net, nonzero_bias=True)
    for p in params:
        p["w"] = np.abs(p["w"]) + np.float32(1e-3)
    obs = np.clip(synth.make_obs(net, batch), -1.0, 1.0)
    bad = np.arange(0, batch, 3)
    obs[bad, 7] = 1e5
    actions, _ = _run_gpu(aq, net, params, obs)
    assert (actions[bad] == np.inf).all()
    assert np.isfinite(np.delete(actions, bad, axis=0)).all()
