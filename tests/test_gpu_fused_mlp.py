"""The general whole-network 8-bit kernel where it can go wrong: LayerNorms over more than 256 features, one feature past a tile
and one short of it, layers that leave wavefronts without a tile, wide last layers, both weight schemes, 8-bit and misaligned
observations, at row counts on both sides of its workgroups' sizes; every stage against the oracle."""
import numpy as np
import pytest
import torch

import gpu_util as U
from paper_1910_01055_amd import synth

pytestmark = pytest.mark.gpu
fc = synth.fc

NETS = {
    "ln263": ([fc(17, 263, "ln_tanh"), fc(263, 163, "relu"), fc(163, 2, "none")], "tanh", "f32"),
    "ln512": ([fc(41, 512, "ln_tanh"), fc(512, 257, "relu"), fc(257, 512, "ln_tanh"), fc(512, 17, "none")], "linear", "f32"),
    "large": ([fc(61, 512, "relu"), fc(512, 511, "none"), fc(511, 490, "relu"), fc(490, 17, "none")], "tanh", "f32"),
    "ln1000": ([fc(65, 1000, "ln_tanh"), fc(1000, 513, "none"), fc(513, 64, "none")], "argmax", "f32"),
    "ln1024": ([fc(3, 1024, "ln_tanh"), fc(1024, 1, "relu"), fc(1, 1024, "relu"), fc(1024, 33, "none")], "tanh", "f32"),
    "ln_one": ([fc(300, 1, "ln_tanh"), fc(1, 700, "ln_tanh"), fc(700, 9, "none")], "tanh", "f32"),
    "wide_last": ([fc(100, 609, "relu"), fc(609, 1000, "none")], "linear", "f32"),
    "wide_argmax": ([fc(257, 31, "ln_tanh"), fc(31, 65, "none")], "argmax", "f32"),
    "u8_long": ([fc(2496, 300, "ln_tanh"), fc(300, 5, "none")], "tanh", "u8"),
    "one_layer": ([fc(261, 40, "none")], "tanh", "f32"),
}
# rows per workgroup and feature tiles per wavefront (in pairs) that the plan gives; (rows, 1): up to 512 wide
VARIANTS = [(name, scheme, batch) for name in NETS for scheme in ("channel_sym_s8", "tensor_asym_u8") for batch in (1, 33)] + [
    ("ln263", "channel_sym_s8", 24577), ("ln263", "tensor_asym_u8", 24577), ("ln512", "channel_sym_s8", 16385),
    ("ln512", "channel_sym_s8", 24700), ("ln512", "tensor_asym_u8", 24577), ("ln512", "tensor_asym_u8", 4097),
    ("large", "channel_sym_s8", 16384), ("large", "channel_sym_s8", 16385), ("large", "tensor_asym_u8", 16385),
    ("ln1000", "channel_sym_s8", 8193), ("ln1000", "tensor_asym_u8", 8193), ("ln1000", "channel_sym_s8", 4097),
    ("ln1000", "tensor_asym_u8", 4097), ("wide_last", "tensor_asym_u8", 8200), ("wide_argmax", "channel_sym_s8", 24600)]


@pytest.mark.parametrize("name,scheme,batch", VARIANTS)
def test_general_kernel_against_the_oracle(aq, name, scheme, batch):
    layers, head, in_type = NETS[name]
    net = synth.small_net(layers, head=head, wscheme=scheme, in_type=in_type)
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    pol, ranges = U.make_oracle(net, params, synth.make_obs(net, 256))
    P, _ = U.gpu_quantize(aq, net, params, ranges)
    P.policy_set_path(1)
    widest = max([l["out"] for l in layers[:-1]], default=0)
    rows, tiles, kind = P.policy_fused_plan(batch)
    assert kind == 0 and tiles == (2 if widest > 512 else 1)
    sym = scheme == "channel_sym_s8"
    want = 16 if batch <= 4096 else (32 if batch <= 8192 else 64) if widest > 512 else \
        (64 if batch > 16384 and sym and name == "large" else 32) if batch <= 24576 else 128 if sym else 64 if widest > 480 else 32
    assert rows == want
    print(f"general kernel {name} {scheme} batch={batch} rows={rows}", flush=True)
    pick = None if batch < 64 else np.unique(np.concatenate([[0, 15, 16, 127, 128, batch - 2, batch - 1],
                                                             np.random.default_rng(5).integers(0, batch, 60)]))
    for misalign in (0, 1):
        actions, t = U.gpu_forward(P, net, obs, misalign=misalign)
        U.compare_forward(net, pol, obs, actions, t, pick)
        plain, _ = U.gpu_forward(P, net, obs, taps=False, misalign=misalign)
        assert np.array_equal(plain, actions, equal_nan=True)
    P.close()


@pytest.mark.parametrize("scheme", ["channel_sym_s8", "tensor_asym_u8"])
@pytest.mark.parametrize("n", [263, 512, 1024])
def test_wide_layernorm_loses_nothing_to_the_layers_launches(aq, n, scheme):
    """LayerNorms of more than 256 features: the tanh values and the codes are no further from the 64-bit ones than those of rows that
    lie in memory (one launch per layer).  Bounds: the values' root mean square error, over 10^7 of them, within 3 %; the number of
    codes off, a count of rare events, within four of its standard deviations."""
    batch = (1 << 24) // n
    net = synth.small_net([fc(61, n, "ln_tanh"), fc(n, 300, "relu"), fc(300, 7, "none")], wscheme=scheme)
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, batch)
    _, ranges = U.make_oracle(net, params, obs[:256])
    P, d = U.gpu_quantize(aq, net, params, ranges)
    m = torch.empty(n, device=U.DEV)
    P.policy_export_layer(0, mult=None, m=m)
    s, z = torch.empty(3, device=U.DEV), torch.empty(3, dtype=torch.int32, device=U.DEV)
    P.policy_export_act_qparams(s, z)
    got = {}
    for path in (1, 2):
        P.policy_set_path(path)
        _, t = U.gpu_forward(P, net, obs)
        x = (t["acc"][0].float() * m).double()
        x -= x.mean(1, keepdim=True)
        x /= torch.sqrt((x * x).mean(1, keepdim=True) + net["ln_eps"])
        want = torch.tanh(x * d[2][0].double() + d[3][0].double())
        code = (torch.round(want / s[1].double()) + z[1]).clamp(0, 255).to(torch.uint8)
        got[path] = float((t["ln_t"][0].double() - want).square().mean().sqrt()), int((code != t["act"][0]).sum())
    print(f"general kernel, LayerNorm of {n}, {scheme}: (rms error, codes off) whole {got[1]}, by layers {got[2]}", flush=True)
    assert got[1][0] <= 1.03 * got[2][0]
    assert got[1][1] <= got[2][1] + 4 * got[2][1] ** 0.5
    P.close()


@pytest.mark.parametrize("n", [200, 700])
def test_a_layernorm_whose_variance_overflows(aq, n):
    """Rows of 1e20 and more: fp32 has no variance for them, its reciprocal root is zero and every value the offset's tanh, from the
    whole-network kernel as from rows in memory."""
    net = synth.small_net([fc(61, n, "ln_tanh"), fc(n, 300, "relu"), fc(300, 7, "none")])
    params = synth.make_params(net, nonzero_bias=True)
    obs = synth.make_obs(net, 100) * np.float32(1e21)
    P, d = U.gpu_quantize(aq, net, params, [(-4e21, 4e21), (-1.0, 1.0), (0.0, 3.0)])
    want = torch.tanh(d[3][0]).expand(100, n)
    for path in (1, 2):
        P.policy_set_path(path)
        _, t = U.gpu_forward(P, net, obs)
        assert torch.isfinite(t["ln_t"][0]).all() and (t["ln_t"][0] - want).abs().max() < 1e-6, path
    P.close()
