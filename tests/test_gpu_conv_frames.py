"""The 8-bit convolutions in one launch at the frames where they can go wrong: rows that are no multiple of 16 bytes, fewer
than four channels, kernel rows that end in the middle of an MFMA's k-step, three and four tiles of features, weights that
do not fit into LDS, maps that share LDS with the frame, more images than workgroups, frames at any address."""
import numpy as np
import pytest

import gpu_util as U
from paper_1910_01055_amd import synth

pytestmark = pytest.mark.gpu
fc, conv = synth.fc, synth.conv


def _net(h, w, c, *layers):
    """layers: (out channels, kernel, stride)"""
    out = []
    for n, k, s in layers:
        out.append(conv(h, w, c, n, k, k, s, "relu"))
        h, w, c = (h - k) // s + 1, (w - k) // s + 1, n
    out += [fc(h * w * c, 40, "relu"), fc(40, 6, "none")]
    return synth.small_net(out, head="argmax", in_type="u8"), len(layers)


NETS = {
    "odd_3": _net(53, 61, 3, (32, 8, 4), (32, 4, 2)),
    "odd_2": _net(54, 67, 2, (16, 8, 4), (32, 4, 2)),
    "odd_1": _net(51, 55, 1, (32, 8, 4), (32, 4, 2), (16, 3, 1)),
    "side_100": _net(100, 100, 4, (32, 8, 4), (32, 4, 2), (16, 3, 1)),
    "kernel_row_48": _net(45, 37, 4, (16, 4, 4), (16, 3, 1), (32, 3, 1)),
    "tiles_3": _net(40, 36, 4, (96, 4, 4), (80, 3, 1)),
    "four_layers": _net(64, 60, 4, (16, 8, 4), (32, 3, 1), (16, 3, 1), (48, 3, 1)),
    "weights_from_l2": _net(33, 33, 16, (128, 3, 1), (16, 3, 1)),
    "ragged_channels": _net(30, 26, 4, (20, 4, 4), (36, 4, 4)),
    # the second map in the frame's place: three layers, and four with that map the larger of the two
    "shared_maps": _net(64, 64, 8, (112, 4, 2), (32, 4, 1), (16, 4, 2)),
    "shared_maps_4": _net(30, 30, 16, (96, 4, 1), (128, 3, 1), (16, 4, 1), (8, 4, 2)),
    # channels that are no multiple of four, and frames of few channels whose windows are whole pieces as they are
    "channels_6": _net(64, 62, 6, (32, 16, 8), (32, 3, 1)),
    "channels_5": _net(50, 49, 5, (16, 16, 16), (16, 2, 1)),
    "one_channel": _net(128, 157, 1, (32, 32, 16), (32, 3, 1)),
}


@pytest.mark.parametrize("name", list(NETS))
@pytest.mark.parametrize("batch", [1, 70, 515])
def test_frames_of_any_size(aq, name, batch):
    print(f"[conv frames] {name} batch={batch}", flush=True)
    net, nc = NETS[name]
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    rows = np.unique([0, batch // 2, max(batch - 260, 0), max(batch - 2, 0), batch - 1])
    pol, ranges = U.make_oracle(net, params, obs[rows])
    P, _ = U.gpu_quantize(aq, net, params, ranges)
    assert P.policy_conv_stack_layers() == nc
    actions, t = U.gpu_forward(P, net, obs)
    U.compare_forward(net, pol, obs, actions, t, rows=rows)
    for misalign in (0, 1, 3):
        plain, _ = U.gpu_forward(P, net, obs, taps=False, misalign=misalign)
        assert np.array_equal(plain, actions)
    P.policy_set_path(3)
    layers, _ = U.gpu_forward(P, net, obs, taps=False)
    assert np.array_equal(layers, actions)
    P.close()
