"""Wide 8-bit layers at many rows (policies wider than the whole-network kernels hold): ragged K and N, LayerNorm rows, a last row
block of one row and of all, both weight schemes, misaligned observations, on both sides of where that kernel begins and ends, also
in front of layers it does not take; every stage against the oracle.  (Which kernel each layer takes: test_host_routes.py.)"""
import numpy as np
import pytest

import gpu_util as U
from paper_1910_01055_amd import synth

pytestmark = pytest.mark.gpu
fc = synth.fc
NETS = {
    "whole": ([fc(128, 2048, "relu"), fc(2048, 1024, "none"), fc(1024, 21, "none")], "tanh"),
    "ragged": ([fc(67, 1300, "relu"), fc(1300, 1043, "ln_tanh"), fc(1043, 37, "none")], "argmax"),
    "ln_first": ([fc(381, 1100, "ln_tanh"), fc(1100, 1031, "relu"), fc(1031, 512, "ln_tanh"), fc(512, 40, "none")], "linear"),
    "2048x3": ([fc(67, 2048, "relu"), fc(2048, 2048, "relu"), fc(2048, 2048, "relu"), fc(2048, 21, "none")], "tanh"),
    "narrow_third": ([fc(67, 2048, "ln_tanh"), fc(2048, 2048, "relu"), fc(2048, 256, "relu"), fc(256, 21, "none")], "tanh"),
    "wide_last": ([fc(67, 2048, "relu"), fc(2048, 1100, "ln_tanh"), fc(1100, 512, "none")], "linear"),
    "narrow_first": ([fc(200, 200, "relu"), fc(200, 1300, "ln_tanh"), fc(1300, 1043, "relu"), fc(1043, 21, "none")], "tanh"),
    "narrow_between": ([fc(20, 1100, "relu"), fc(1100, 200, "relu"), fc(200, 1030, "relu"), fc(1030, 5, "none")], "tanh"),
}


CASES = [(name, batch) for name in ("whole", "ragged", "ln_first", "narrow_between") for batch in (449, 450, 513, 1024)] + [
    ("2048x3", 8128), ("2048x3", 8150), ("narrow_third", 960), ("narrow_third", 961), ("narrow_third", 1300), ("wide_last", 1300),
    ("wide_last", 4500), ("narrow_between", 3000), ("narrow_first", 640), ("narrow_first", 1300)]


@pytest.mark.parametrize("name,batch", CASES)
@pytest.mark.parametrize("scheme", ["channel_sym_s8", "tensor_asym_u8"])
def test_wide_layers_at_many_rows(aq, name, scheme, batch):
    print(f"[rows layer] {name} {scheme} batch={batch}", flush=True)
    net = synth.small_net(NETS[name][0], head=NETS[name][1], wscheme=scheme)
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    pol, ranges = U.make_oracle(net, params, obs[:256])
    P, _ = U.gpu_quantize(aq, net, params, ranges)
    rows = np.unique(np.concatenate([[0, 15, 16, 63, 64, batch - 2, batch - 1], np.random.default_rng(6).integers(0, batch, 40)]))
    for misalign in (0, 1):
        actions, t = U.gpu_forward(P, net, obs, misalign=misalign)
        U.compare_forward(net, pol, obs, actions, t, rows)
        plain, _ = U.gpu_forward(P, net, obs, taps=False, misalign=misalign)
        assert np.array_equal(plain, actions, equal_nan=True)
    P.close()
