"""The fp32 actor's kernels against the CPU oracle at the sizes where they can go wrong: every tile of the per-layer
kernel with ragged rows, features and K, convolutions whose windows allow no 16-byte loads, and the whole-MLP kernel's
layer widths, heads and row counts."""
import numpy as np
import pytest
import torch

from oracle import policy as O
from paper_1910_01055_amd import synth
import gpu_util as U

pytestmark = pytest.mark.gpu
fc, conv = synth.fc, synth.conv


def _cases():
    small = lambda *a, **k: synth.small_net(*a, **k)  # noqa: E731
    return {
        # one launch: widths around whole stages and feature tiles, each head, both input types
        "mlp_tanh": (small([fc(17, 33, "relu"), fc(33, 47, "none"), fc(47, 6, "none")]), [1, 15, 17, 300]),
        "mlp_ln": (small([fc(111, 400, "ln_tanh"), fc(400, 300, "relu"), fc(300, 8, "none")]), [1, 97]),
        "mlp_argmax": (small([fc(5, 16, "relu"), fc(16, 64, "relu"), fc(64, 18, "none")], head="argmax"), [1, 33]),
        "mlp_wide_head": (small([fc(31, 64, "relu"), fc(64, 100, "none")], head="linear"), [1, 40]),
        "mlp_wide_argmax": (small([fc(31, 64, "relu"), fc(64, 70, "none")], head="argmax"), [50]),
        "mlp_u8": (small([fc(48, 65, "relu"), fc(65, 5, "none")], head="linear", in_type="u8"), [3, 64]),
        "mlp_single": (small([fc(50, 37, "none")]), [19]),
        "mlp_two_tiles": (small([fc(20, 256, "relu"), fc(256, 21, "none")]), [8193 + 16]),  # 32 rows per workgroup
        # LayerNorms on either side of the widths that a wavefront holds in registers, one and two row tiles per workgroup
        **{"mlp_ln_%d" % n: (small([fc(20, n, "ln_tanh"), fc(n, 7, "none")]), bs)
           for n, bs in ((128, [40]), (129, [40, 4097]), (300, [4096, 4097]), (512, [40]), (513, [40]))},
        # a launch per layer: wide layers, few and many rows
        "layers_few_rows": (small([fc(67, 1300, "ln_tanh"), fc(1300, 1300, "relu"), fc(1300, 21, "none")]), [1, 16, 17, 70]),
        "layers_many_rows": (small([fc(70, 1300, "relu"), fc(1300, 130, "none"), fc(130, 66, "none")], head="argmax"), [513, 2100]),
        # ... on the two largest tiles, of 64 features x 128 rows and of 64 x 64
        "layers_tile_64x128": (small([fc(67, 600, "relu"), fc(600, 2047, "none"), fc(2047, 3, "none")]), [1003]),
        "layers_tile_64x64": (small([fc(70, 1300, "relu"), fc(1300, 190, "none"), fc(190, 4, "none")]), [5437]),
        "conv": (small([conv(20, 20, 4, 33, 8, 8, 4, "relu"), conv(4, 4, 33, 20, 2, 2, 1, "none"), fc(180, 24, "relu"), fc(24, 5, "none")],
                       head="linear", in_type="u8", init="he_normal"), [1, 70]),
        "conv_odd_window": (small([conv(9, 10, 3, 5, 3, 2, 2, "relu"), conv(4, 5, 5, 7, 3, 3, 1, "relu"), fc(42, 11, "none")],
                                  head="linear", in_type="u8", init="he_normal"), [1, 200]),
        "conv_f32": (small([conv(12, 12, 3, 64, 4, 4, 2, "relu"), conv(5, 5, 64, 65, 3, 3, 1, "relu"), fc(585, 4, "none")],
                           head="tanh", init="he_normal"), [90]),
    }


@pytest.mark.parametrize("name,batch", [(n, b) for n, (_, bs) in _cases().items() for b in bs])
def test_fp32_actor_and_ranges(aq, name, batch):
    net = _cases()[name][0]
    print(f"[fp32] {name} batch={batch}", flush=True)
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    if net["in_type"] == "u8":  # frames are consumed as raw codes: keep the activations near one
        params[0]["w"] /= 255.0
    ref, ranges = O.OraclePolicy(net).forward_fp32(params, obs)
    P = aq.Policy(net)
    w, b, g, be = U.upload_params(params)
    P.policy_set_params_fp32(w, b, g, be)
    d_obs = U.to_dev(obs)
    argmax = net["head"] == "argmax"
    out = torch.full((batch,) if argmax else (batch, synth.action_dim(net)), -7, dtype=torch.int32 if argmax else torch.float32,
                     device=U.DEV)
    passed = torch.empty_like(out)
    P.policy_forward_fp32(d_obs, out)
    P.policy_forward_fp32_params(w, b, g, be, d_obs, passed)
    for _ in range(2):  # (a calibration leaves its accumulators ready for the next)
        got = np.array(P.calibrate_fp32(d_obs))
        want = np.array(ranges)
        assert (np.abs(got - want) <= 1e-5 * np.abs(want) + 1e-6).all()
    torch.cuda.synchronize()
    assert torch.equal(out, passed)
    if argmax:
        assert (out.cpu().numpy() == ref).mean() >= 0.99
    else:
        assert U.close(out.cpu().numpy(), ref).all()
    P.close()


def test_the_cases_reach_every_tile(aq):
    """... of the per-layer kernel, and both forms of the whole-policy kernel."""
    rows, tiles = set(), set()
    for net, batches in _cases().values():
        P = aq.Policy(net)
        for batch in batches:
            r, t = P.policy_fp32_plan(batch)
            rows.add(r)
            tiles.update(t)
        P.close()
    assert rows == {0, 16, 32}
    assert tiles == {(64, 128), (32, 128), (64, 64), (32, 32), (16, 32), (16, 16)}


def test_two_row_tiles_per_workgroup_from_the_second_round_on(aq):
    P = aq.Policy(synth.small_net([fc(20, 256, "relu"), fc(256, 21, "none")]))
    assert [P.policy_fp32_plan(b)[0] for b in (1, 4096, 4097, 8193)] == [16, 16, 32, 32]
    P.close()


def test_batches_beyond_a_grid_of_whole_policy_workgroups_go_layer_by_layer(aq):
    """A grid holds fewer than 2^32 threads: 1024 for each 32 rows of the whole-policy kernel, 512 for each 128 rows of a
    layer's largest tile.  (Plans only: such a batch's observations are gigabytes.)"""
    P = aq.Policy(synth.small_net([fc(4, 64, "relu"), fc(64, 2, "none")]))
    assert P.policy_fp32_plan((1 << 27) - 32)[0] == 32
    for batch in ((1 << 27) - 31, 1 << 27, (1 << 30) - 128):
        rows, tiles = P.policy_fp32_plan(batch)
        assert rows == 0
        assert all(-(-batch // r) * 512 < 1 << 32 for _, r in tiles), tiles
    P.close()


def test_fp32_calibration_of_a_smaller_batch_forgets_the_larger_ones_ranges(aq):
    net = synth.net_config("cfg4")
    params = synth.make_params(net)
    P = aq.Policy(net)
    P.policy_set_params_fp32(*U.upload_params(params))
    obs = U.to_dev(synth.make_obs(net, 12))
    first = P.calibrate_fp32(obs[:2])
    P.calibrate_fp32(obs)
    assert P.calibrate_fp32(obs[:2]) == first
    P.close()


def test_fp32_forward_on_passed_parameters_is_captured_after_reserve(aq):
    """After a reserve the first call of the forward that takes its parameters may be one into a graph."""
    net = synth.small_net([fc(17, 300, "relu"), fc(300, 1100, "relu"), fc(1100, 6, "none")])
    params = synth.make_params(net, nonzero_bias=True)
    dev = U.upload_params(params)
    obs, out = U.to_dev(synth.make_obs(net, 40)), torch.zeros(40, 6, device=U.DEV)
    P = aq.Policy(net)
    P.policy_reserve(40)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        P.policy_forward_fp32_params(*dev, obs, out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        replayed = out.clone()
        P.policy_forward_fp32_params(*dev, obs, out)
        torch.cuda.synchronize()
        assert torch.equal(replayed, out)
    assert U.close(replayed.cpu().numpy(), O.OraclePolicy(net).forward_fp32(params, synth.make_obs(net, 40))[0]).all()
    P.close()


def test_fp32_weights_cost_memory_only_where_they_are_used(aq):
    """A policy that has run nothing in fp32 holds its 8-bit weights and constants, about a byte per weight."""
    net = synth.small_net([fc(64, 2048, "relu"), fc(2048, 2048, "relu"), fc(2048, 2048, "relu"), fc(2048, 8, "none")])
    params = synth.make_params(net, nonzero_bias=True)
    weights = sum(p["w"].size for p in params)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    policies = [aq.Policy(net) for _ in range(8)]
    held = before - torch.cuda.mem_get_info()[0]
    assert held < 8 * 1.6 * weights, held / (8 * weights)
    for P in policies:
        P.close()


def test_first_fp32_forward_on_passed_parameters_under_capture(aq):
    """The first call allocates its packed weights: a policy that needs no other buffers may make it into a graph."""
    net = synth.small_net([fc(17, 300, "relu"), fc(300, 200, "ln_tanh"), fc(200, 6, "none")])
    params = synth.make_params(net, nonzero_bias=True)
    dev = U.upload_params(params)
    obs, out, want = U.to_dev(synth.make_obs(net, 40)), torch.zeros(40, 6, device=U.DEV), torch.zeros(40, 6, device=U.DEV)
    P = aq.Policy(net)
    assert P.policy_fp32_plan(40)[0] == 16
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        P.policy_forward_fp32_params(*dev, obs, out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        P.policy_forward_fp32_params(*dev, obs, want)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    assert U.close(out.cpu().numpy(), O.OraclePolicy(net).forward_fp32(params, synth.make_obs(net, 40))[0]).all()
    P.close()


@pytest.mark.parametrize("K,N", [(67, 1300), (3136, 512), (3100, 70)])
@pytest.mark.parametrize("rows", [1, 40, 700, 4100])
def test_an_infinite_weight_stays_infinite_in_the_per_layer_kernel(aq, K, N, rows):
    """A diverged policy: one infinite weight among the last 16 inputs of a layer whose K ends inside a stage.  The unit is
    +infinity on positive inputs, in the actions and in the calibrated ranges; nothing becomes NaN."""
    net = synth.small_net([fc(K, N, "relu"), fc(N, 5, "none")], head="linear")
    print(f"[fp32 inf] K={K} N={N} rows={rows}", flush=True)
    params = synth.make_params(net, nonzero_bias=True)
    params[0]["w"][N // 2, K - 3] = np.inf
    obs = np.abs(synth.make_obs(net, rows)) + np.float32(0.01)
    hidden = np.maximum(obs.astype(np.float64) @ params[0]["w"].T.astype(np.float64) + params[0]["b"], 0.0)
    want = hidden @ params[1]["w"].T.astype(np.float64) + params[1]["b"]
    assert np.isinf(want).all()
    P = aq.Policy(net)
    P.policy_set_params_fp32(*U.upload_params(params))
    out = torch.zeros(rows, 5, device=U.DEV)
    P.policy_forward_fp32(U.to_dev(obs), out)
    ranges = P.calibrate_fp32(U.to_dev(obs))
    assert np.array_equal(out.cpu().numpy(), want.astype(np.float32))
    assert ranges[1][1] == np.inf and ranges[1][0] == 0.0 and np.isfinite(ranges[0]).all()
    P.close()
