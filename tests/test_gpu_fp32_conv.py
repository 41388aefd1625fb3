"""The fp32 convolutions in one launch: frames whose rows are no multiple of four bytes, few channels, K that ends inside a
k-step of 32, one to four layers, every split of positions and K, more images than CUs; and values whose bf16 parts would
leave bf16's range, which take the fp32 instructions."""
import numpy as np
import pytest
import torch

from oracle import policy as O
from paper_1910_01055_amd import synth
import gpu_util as U

pytestmark = pytest.mark.gpu
fc, conv = synth.fc, synth.conv


def _net(h, w, c, *layers):
    """layers: (out channels, kernel, stride)"""
    out = []
    for n, k, s in layers:
        out.append(conv(h, w, c, n, k, k, s, "none" if len(out) == 1 else "relu"))
        h, w, c = (h - k) // s + 1, (w - k) // s + 1, n
    out += [fc(h * w * c, 24, "relu"), fc(24, 6, "none")]
    return synth.small_net(out, head="linear", in_type="u8", init="he_normal")


NETS = {
    "usual": _net(84, 84, 4, (32, 8, 4), (64, 4, 2), (64, 3, 1)),
    "side_99": _net(99, 99, 4, (32, 8, 4), (64, 4, 2), (64, 3, 1)),
    "odd_3_channels": _net(53, 61, 3, (16, 8, 4), (32, 4, 2), (32, 3, 1)),
    "one_channel": _net(52, 55, 1, (16, 8, 4), (32, 4, 2), (32, 3, 1)),
    "one_layer": _net(40, 36, 4, (20, 4, 4)),
    "ragged_features": _net(30, 26, 4, (24, 4, 2), (40, 3, 2), (12, 3, 1)),
    "four_layers": _net(50, 44, 4, (16, 4, 2), (16, 3, 2), (128, 3, 1), (8, 2, 1)),
}


def _run(aq, net, params, obs, one_launch=True):
    P = aq.Policy(net)
    dev = U.upload_params(params)
    P.policy_set_params_fp32(*dev)
    assert (P.policy_fp32_plan(len(obs))[1][0][0] == 0) == one_launch
    d_obs = U.to_dev(obs)
    out = torch.zeros(len(obs), synth.action_dim(net), device=U.DEV)
    passed = torch.empty_like(out)
    P.policy_forward_fp32(d_obs, out)
    P.policy_forward_fp32_params(*dev, d_obs, passed)
    ranges = np.array(P.calibrate_fp32(d_obs))
    torch.cuda.synchronize()
    assert torch.equal(out, passed) or not torch.isfinite(out).all()
    P.close()
    return out.cpu().numpy(), ranges


def _exact(net, params, obs):
    """The actions in 64 bits, and the range of every layer's input."""
    x, ranges = obs.astype(np.float64), []
    for l, p in zip(net["layers"], params):
        ranges.append((x.min(), x.max()))
        w = p["w"].astype(np.float64)
        if l["kind"] == "conv":
            v = np.lib.stride_tricks.sliding_window_view(x, (l["kh"], l["kw"]), (1, 2))[:, ::l["stride"], ::l["stride"]]
            n, oh, ow = v.shape[:3]
            w = w.reshape(l["out_c"], l["kh"], l["kw"], -1).transpose(0, 3, 1, 2).reshape(l["out_c"], -1)
            x = (v.reshape(n * oh * ow, -1) @ w.T + p["b"]).reshape(n, oh, ow, -1)
        else:
            x = x.reshape(len(x), -1) @ w.T + p["b"]
        if l["act"] == "relu":
            x = np.where(x > 0.0, x, 0.0)  # (a NaN becomes 0, as in the library)
    return x, np.array(ranges)


# one image: the layers' own launches but for the smallest frames; then one launch, the second time with a second round of images
# (a single small convolution is faster layer by layer there)
@pytest.mark.parametrize("name,batch", [(n, b) for n in NETS for b in {"one_layer": (1, 256), "odd_3_channels": (1, 70, 400)}.get(n, (1, 70, 310))])
def test_fp32_convolutions_in_one_launch(aq, name, batch):
    print(f"[fp32 conv] {name} batch={batch}", flush=True)
    net = NETS[name]
    params = synth.make_params(net, nonzero_bias=True)
    params[0]["w"] /= 255.0
    obs = synth.make_obs(net, batch)
    out, ranges = _run(aq, net, params, obs, batch > 1 or name in ("odd_3_channels", "one_channel", "ragged_features"))
    want, ref = _exact(net, params, obs)
    # fp32: 2^-24 a rounding, some 5 to 20 of them along a path, in random directions
    assert np.abs(out - want).max() <= 2e-6 * np.abs(want).max()
    assert (ranges[0] == [obs.min(), obs.max()]).all()
    assert (np.abs(ranges - ref) <= 1e-5 * np.abs(ref) + 1e-6).all()
    # a subset's range lies within the batch's
    _, few = O.OraclePolicy(net).forward_fp32(params, obs[[0, batch - 1]])
    few = np.array(few)
    slack = 1e-5 * np.abs(few) + 1e-6
    assert (ranges[:, 0] <= few[:, 0] + slack[:, 0]).all() and (ranges[:, 1] >= few[:, 1] - slack[:, 1]).all()


@pytest.mark.parametrize("layer,value", [(0, np.inf), (1, np.inf), (2, -np.inf), (1, np.nan), (0, 3.4e38), (2, 1e-38)])
def test_weights_outside_of_the_split_range(aq, layer, value):
    """An infinite weight on positive inputs makes its unit infinite and nothing NaN, as in plain fp32; a value that would round
    to infinity in bf16 stays finite; one below 2^-100 keeps its place."""
    net = NETS["odd_3_channels"]
    params = synth.make_params(net, nonzero_bias=False)
    params[0]["w"] /= 255.0
    for p in params:
        p["w"] = np.abs(p["w"])
    if value == 3.4e38:
        params[0]["w"][3] = 0.0
    params[layer]["w"].reshape(params[layer]["w"].shape[0], -1)[3, 5] = value
    obs = np.maximum(synth.make_obs(net, 52), 1)
    if value == 3.4e38:
        obs[:] = 1  # (the unit is exactly this weight)
        params[1]["w"] *= np.float32(1e-20)
    out, ranges = _run(aq, net, params, obs)
    with np.errstate(invalid="ignore"):
        want, _ = _exact(net, params, obs)
    f = np.isfinite(want)
    assert np.array_equal(np.isnan(out), np.isnan(want)) and np.array_equal(out[~f & ~np.isnan(want)], want[~f & ~np.isnan(want)])
    assert np.allclose(out[f], want[f], rtol=1e-5)
    assert ranges[layer + 1][1] == value or value != np.inf


def test_scales_far_from_one(aq):
    """Weights of one layer scaled down and the next one's scaled up by 2^115: the maps between lie below 2^-100."""
    net = NETS["usual"]
    params = synth.make_params(net, nonzero_bias=False)
    params[0]["w"] /= 255.0
    obs = synth.make_obs(net, 70)
    want, _ = _run(aq, net, params, obs)
    params[0]["w"] *= np.float32(2.0 ** -100)
    params[1]["w"] *= np.float32(2.0 ** -15)
    params[2]["w"] *= np.float32(2.0 ** 115)
    got, _ = _run(aq, net, params, obs)
    assert np.abs(got - want).max() <= 4e-6 * np.abs(want).max()
