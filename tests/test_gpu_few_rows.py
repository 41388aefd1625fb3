"""The few-row layer kernel at the edges of its tiles: 16 x 16, 32 x 16 and 32 x 32 outputs, shares of K that are empty,
odd and longer than what is in flight, rows that are no multiple of 16, and maps in operand order between its layers."""
import numpy as np
import pytest

import gpu_util as U
import test_gpu_fp16 as H
from paper_1910_01055_amd import synth

pytestmark = pytest.mark.gpu
fc = synth.fc


def _net(name):
    return {
        # K of 37 and 300 (no whole pieces of 16), widths whose last tile of 16 is ragged, an argmax over one tile of 16
        "odd_argmax16": synth.small_net([fc(37, 300, "relu"), fc(300, 75, "none"), fc(75, 11, "none")], head="argmax"),
        # the last half of a pair of 32-k tiles missing, an argmax over two tiles, a LayerNorm between two layers
        "ln_argmax32": synth.small_net([fc(96, 160, "relu"), fc(160, 96, "ln_tanh"), fc(96, 32, "none")], head="argmax"),
        # a K beyond eight k-steps of 64 per wave
        "long_k": synth.small_net([fc(300, 4500, "relu"), fc(4500, 130, "none"), fc(130, 20, "none")], head="linear"),
        "odd_asym": synth.small_net([fc(50, 500, "relu"), fc(500, 333, "none"), fc(333, 40, "none")], head="tanh",
                                    wscheme="tensor_asym_u8"),
        "u8_rows": synth.small_net([fc(150, 80, "relu"), fc(80, 50, "none")], head="tanh", in_type="u8"),
    }[name]


@pytest.mark.parametrize("name,batches", [("odd_argmax16", (1, 16, 17, 333, 1700)), ("ln_argmax32", (2, 31, 900)),
                                          ("long_k", (1, 40, 500)), ("odd_asym", (1, 15, 260, 700)), ("u8_rows", (5, 48, 2000))])
def test_few_row_layers_against_the_oracle(aq, name, batches):
    net = _net(name)
    params = synth.make_params(net, nonzero_bias=True)
    for batch in batches:
        print(f"few_rows {name} batch={batch}", flush=True)
        obs = synth.make_obs(net, batch)
        pol, ranges = U.make_oracle(net, params, obs[:256])
        P, _ = U.gpu_quantize(aq, net, params, ranges)
        P.policy_set_path(2)
        actions, taps = U.gpu_forward(P, net, obs)
        rows = np.unique(np.concatenate([[0, batch // 2, batch - 1], np.random.default_rng(3).integers(0, batch, 60)]))
        U.compare_forward(net, pol, obs, actions, taps, rows)
        plain, _ = U.gpu_forward(P, net, obs, taps=False)
        assert np.array_equal(plain, actions)
        P.close()


@pytest.mark.parametrize("batch", [1, 16, 33, 270])
@pytest.mark.parametrize("odd,head", [(True, "tanh"), (True, "argmax"), (False, "linear")])
def test_fp16_few_row_layers_against_the_oracle(aq, odd, head, batch):
    """The half-precision counterpart: rows of no whole pieces of eight values behind fp32 observations, an argmax over two tiles of
    16, K beyond eight k-steps of 32 per wave.  (Without intermediate outputs, maps between the layers in operand order.)"""
    print(f"[fp16 few rows] {odd} {head} batch={batch}", flush=True)
    if odd:
        layers = [fc(67, 1099, "relu"), fc(1099, 1037, "none"), fc(1037, 18 if head == "argmax" else 33, "none")]
    else:
        layers = [fc(300, 2400, "relu"), fc(2400, 136, "relu"), fc(136, 16, "none")]
    net = synth.small_net(layers, head=head)
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    P = aq.Policy(net)
    P.convert_params_fp16(*U.upload_params(params))
    assert P.policy_fp16_plan(batch) == 0  # a launch per layer
    P.close()
    actions, outs = H._run_gpu(aq, net, params, obs)
    H._check(net, params, obs, actions, outs, end_to_end=False)


@pytest.mark.parametrize("channels,batches", [(8, (3968, 3969)), (9, (9984, 9985))])
def test_fp16_layers_at_the_last_rows_of_the_few_row_kernel(aq, channels, batches):
    """... and the first of the tiled one: a hidden layer of 200 inputs, and of 225, behind a convolution."""
    net = synth.small_net([synth.conv(12, 12, 2, channels, 4, 4, 2, "relu"), fc(25 * channels, 100, "relu"), fc(100, 11, "none")],
                          head="argmax", in_type="u8", init="he_normal")
    params = synth.make_params(net, nonzero_bias=True)
    for batch in batches:
        print(f"[fp16 few rows] {channels} batch={batch}", flush=True)
        obs = synth.make_obs(net, batch)
        actions, outs = H._run_gpu(aq, net, params, obs)
        rows = np.unique(np.concatenate([[0, 15, 16, 31, 32, batch - 2, batch - 1], np.random.default_rng(3).integers(0, batch, 40)]))
        H._check(net, params, obs[rows], actions[rows], [o.reshape(batch, -1)[rows] for o in outs], end_to_end=False)


def test_wide_policies_at_few_rows_take_the_layers_launches(aq):
    """Which plan an MLP that fits the whole-network kernels takes on either side of the rule, and the same integers from both
    plans, from a second stream while the first is busy, and from more streams than there are pairs of maps."""
    import torch
    net = synth.small_net([fc(67, 1000, "relu"), fc(1000, 720, "none"), fc(720, 21, "none")], head="tanh")
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, 513)
    _, ranges = U.make_oracle(net, params, obs[:256])
    P, _ = U.gpu_quantize(aq, net, params, ranges)
    for batch, layers in ((1, True), (16, True), (250, True), (513, False)):
        assert (P.policy_fused_plan(batch)[0] == 0) == layers, batch
        P.policy_set_path(1)
        whole, _ = U.gpu_forward(P, net, obs[:batch], taps=False)
        P.policy_set_path(0)
        assert np.array_equal(U.gpu_forward(P, net, obs[:batch], taps=False)[0], whole)
    P.policy_set_path(1)
    want = U.gpu_forward(P, net, obs[:250], taps=False)[0]
    P.policy_set_path(0)
    d_obs = aq.to_dev(obs[:250])
    outs, streams = [], [torch.cuda.Stream() for _ in range(6)]
    torch.cuda.synchronize()
    for rep in range(8):
        for s in streams:
            with torch.cuda.stream(s):
                y = torch.zeros((250, 21), device="cuda:0")
                P.policy_forward_int8(d_obs, y)
                outs.append(y)
    torch.cuda.synchronize()
    assert all(np.array_equal(y.cpu().numpy(), want) for y in outs)
    # the handle that names another stream in every thread
    with torch.cuda.stream(torch.cuda.ExternalStream(2)):
        y = torch.zeros((250, 21), device="cuda:0")
        P.policy_forward_int8(d_obs, y)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), want)
    P.close()
    # per-tensor weights, exploration behind the layers
    net = synth.small_net([fc(40, 1024, "relu"), fc(1024, 1024, "relu"), fc(1024, 30, "none")], head="tanh", wscheme="tensor_asym_u8")
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, 200)
    _, ranges = U.make_oracle(net, params, obs)
    P, _ = U.gpu_quantize(aq, net, params, ranges)
    assert P.policy_fused_plan(200)[0] == 0
    d_obs, sigma = aq.to_dev(obs), torch.full((200,), 0.1, device="cuda:0")
    got = []
    for path in (0, 1):
        P.policy_set_path(path)
        y = torch.zeros((200, 30), device="cuda:0")
        P.policy_step_int8(d_obs, y, 5, 3, sigma=sigma)
        got.append(y.cpu().numpy())
    assert np.array_equal(got[0], got[1])
    P.close()


@pytest.mark.parametrize("actions", [16, 17, 32, 33])
def test_wide_argmax_policies_at_few_rows(aq, actions):
    """The layers' launches find the index in the last of them, without logits in memory: up to 32 outputs, which one workgroup
    holds; 33 keep the whole-network kernel.  The same integers from both plans, with the logits too, and with exploration."""
    import torch
    net = synth.small_net([fc(40, 1024, "relu"), fc(1024, 1024, "none"), fc(1024, actions, "none")], head="argmax")
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, 200)
    pol, ranges = U.make_oracle(net, params, obs)
    P, _ = U.gpu_quantize(aq, net, params, ranges)
    for batch in (1, 33, 200):
        print(f"few_rows argmax {actions} batch={batch}", flush=True)
        d_obs, got = aq.to_dev(obs[:batch]), []
        P.policy_set_path(0)
        assert (P.policy_fused_plan(batch)[0] == 0) == (actions <= 32)
        for path in (0, 1):
            P.policy_set_path(path)
            plain, _ = U.gpu_forward(P, net, obs[:batch], taps=False)
            with_taps, taps = U.gpu_forward(P, net, obs[:batch])
            assert np.array_equal(plain, with_taps)
            only_y = torch.zeros((batch, actions), device=U.DEV)
            act = torch.full((batch,), -7, dtype=torch.int32, device=U.DEV)
            P.policy_forward_int8(d_obs, act, {"y": only_y})
            explored = torch.full((batch,), -7, dtype=torch.int32, device=U.DEV)
            P.policy_step_int8(d_obs, explored, 11, 4, epsilon=0.4)
            got.append([plain, act.cpu().numpy(), only_y.cpu().numpy(), explored.cpu().numpy()])
            U.compare_forward(net, pol, obs[:batch], with_taps, taps)
        for a, b in zip(*got):
            assert np.array_equal(a, b)
        assert batch == 1 or (got[0][3] != got[0][0]).any()
    P.close()


def test_captured_and_allocation_free_forwards_of_a_wide_policy(aq):
    """Both keep the whole-network kernel: a graph's replays and the static entry point beside eager forwards on the layers'
    launches, on the same stream and another, give the same actions."""
    import torch
    net = synth.small_net([fc(67, 1024, "relu"), fc(1024, 1024, "relu"), fc(1024, 21, "none")], head="tanh")
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, 96)
    pol, ranges = U.make_oracle(net, params, obs)
    P, _ = U.gpu_quantize(aq, net, params, ranges)
    assert P.policy_fused_plan(96)[0] == 0
    d_obs, side = aq.to_dev(obs), torch.cuda.Stream()
    want = torch.zeros((96, 21), device=U.DEV)
    P.policy_forward_int8(d_obs, want)
    assert U.close(want.cpu().numpy(), pol.forward_int8(obs)["actions"]).all()
    graph, y = torch.cuda.CUDAGraph(), torch.zeros((96, 21), device=U.DEV)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        P.policy_forward_int8(d_obs, y)
    for _ in range(4):
        y.zero_()
        eager, static, other = (torch.zeros((96, 21), device=U.DEV) for _ in range(3))
        torch.cuda.synchronize()
        graph.replay()
        P.policy_forward_int8(d_obs, eager)
        P.policy_forward_int8_static(d_obs, static)
        with torch.cuda.stream(side):
            P.policy_forward_int8(d_obs, other)
        torch.cuda.synchronize()
        for got in (y, eager, static, other):
            assert torch.equal(got, want)
    P.close()
