"""LayerNorm layers that run on their own, in the three precisions, at the edges of the forms their kernels take: one or four
wavefronts to a row, one, two or four pieces a thread, rows of no whole pieces, and rows longer than any form holds."""
import numpy as np
import pytest
import torch

import gpu_util as U
import test_gpu_fp16 as H
from oracle import policy as O
from paper_1910_01055_amd import synth

pytestmark = pytest.mark.gpu
fc = synth.fc
# one row to four wavefronts up to 1023 rows of up to 1024 values (short ones leave wavefronts without a value), one wavefront each
# behind that, four for longer ones
SHAPES = [(1, 3), (100, 9), (193, 5), (256, 3), (257, 17), (1024, 1023), (1024, 1024), (1021, 1025), (255, 1030), (512, 1100), (1025, 5),
          (1028, 1100), (2048, 16), (2047, 16), (2052, 7), (4096, 5), (4097, 5)]


def _net(n):
    return synth.small_net([fc(37, n, "ln_tanh"), fc(n, 40, "relu"), fc(40, 5, "none")])


@pytest.mark.parametrize("n,batch", SHAPES)
def test_int8(aq, n, batch):
    print(f"[ln rows] int8 {n} x {batch}", flush=True)
    net = _net(n)
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    pol, ranges = U.make_oracle(net, params, obs[:256])
    P, _ = U.gpu_quantize(aq, net, params, ranges)
    P.policy_set_path(2)  # a launch per layer
    actions, taps = U.gpu_forward(P, net, obs)
    rows = np.unique(np.concatenate([[0, batch // 2, batch - 1], np.random.default_rng(3).integers(0, batch, 40)]))
    U.compare_forward(net, pol, obs, actions, taps, rows)
    plain, _ = U.gpu_forward(P, net, obs, taps=False)
    assert np.array_equal(plain, actions)
    P.close()


@pytest.mark.parametrize("n,batch", [s for s in SHAPES if s[0] > 1024])  # (the others run as one launch)
def test_fp16(aq, n, batch):
    print(f"[ln rows] fp16 {n} x {batch}", flush=True)
    net = _net(n)
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    actions, outs = H._run_gpu(aq, net, params, obs)
    H._check(net, params, obs, actions, outs, end_to_end=False)


@pytest.mark.parametrize("hidden", [1400, 1022, 100, 1])  # four wavefronts to a row, in whole pieces and not, with idle ones, and one
@pytest.mark.parametrize("batch", [900, 1030])
def test_fp16_behind_a_wide_layer(aq, hidden, batch):
    net = synth.small_net([fc(20, 1400, "relu"), fc(1400, hidden, "ln_tanh"), fc(hidden, 9, "none")])
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    actions, outs = H._run_gpu(aq, net, params, obs)
    H._check(net, params, obs, actions, outs, end_to_end=False)


@pytest.mark.parametrize("n,batch", SHAPES)
def test_fp32(aq, n, batch):
    print(f"[ln rows] fp32 {n} x {batch}", flush=True)
    net = synth.small_net([fc(37, n, "ln_tanh"), fc(n, 1300, "relu"), fc(1300, 5, "none")])  # (a layer too wide for one launch)
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    ref, ranges = O.OraclePolicy(net).forward_fp32(params, obs)
    P = aq.Policy(net)
    w, b, g, be = U.upload_params(params)
    P.policy_set_params_fp32(w, b, g, be)
    d_obs = U.to_dev(obs)
    out, passed = torch.empty(batch, 5, device=U.DEV), torch.empty(batch, 5, device=U.DEV)
    P.policy_forward_fp32(d_obs, out)
    # gains and offsets of the caller's own that start at any float
    shift = [None if t is None else torch.cat([t.new_zeros(1), t])[1:] for t in g], [None if t is None else torch.cat([t.new_zeros(1), t])[1:] for t in be]
    P.policy_forward_fp32_params(w, b, *shift, d_obs, passed)
    got, want = np.array(P.calibrate_fp32(d_obs)), np.array(ranges)
    torch.cuda.synchronize()
    assert (np.abs(got - want) <= 1e-5 * np.abs(want) + 1e-6).all()
    assert U.close(out.cpu().numpy(), ref).all() and U.close(passed.cpu().numpy(), ref).all()
    P.close()
