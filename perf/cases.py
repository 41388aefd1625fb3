"""The work that actors and learners have this library do, as cases with stated sizes.

An actor runs the policy on the observations at hand, in 8 bits (the path the library is for), in half precision or
in fp32.  A learner calibrates the activation ranges on a batch from replay and hands the quantized policy to its
actors; a learner that only broadcasts weights quantizes single tensors.  Every case goes through the binding, one
call at a time on torch's current stream, as a program that uses the library does.
"""
import math

import torch

from paper_1910_01055_amd import binding as aq
from paper_1910_01055_amd import synth

DEV = "cuda:0"
CALIBRATION_ROWS = 512
CALIBRATION_FRAMES = 32


def _mlp(do, bits, inputs, widths, actions, batch, ln=False, scheme="channel_sym_s8", explore=False, wbits=8):
    """A fully connected policy of continuous control: tanh actions, LayerNorm + tanh behind the first layer if `ln`."""
    w = list(widths) + [0, 0, 0]
    return {"do": do, "bits": bits, "net": "mlp", "inputs": inputs, "width1": w[0], "width2": w[1], "width3": w[2],
            "actions": actions, "batch": batch, "ln": ln, "scheme": scheme, "explore": explore, "wbits": wbits}


def _frames(do, bits, side, stack, channels, hidden, actions, batch):
    """A value network on stacks of 8-bit frames: three convolutions, one hidden layer, a value for each action."""
    return {"do": do, "bits": bits, "net": "frames", "side": side, "stack": stack, "channels": channels, "width1": hidden,
            "actions": actions, "batch": batch, "scheme": "channel_sym_s8", "explore": False, "wbits": 8}


def listed():
    return [
        # one actor process with one environment, per-tensor weights: nothing but latency
        dict(_mlp("act", 8, 17, (256, 256), 6, 1, scheme="tensor_asym_u8"), name="act8 small b1"),
        # the usual vectorised actor: LayerNorm policy, Gaussian exploration with a sigma for each actor
        dict(_mlp("act", 8, 67, (256, 256, 256), 21, 4096, ln=True, explore=True), name="act8 control b4096"),
        # the same policy on as many environments as a GPU simulator steps at once
        dict(_mlp("act", 8, 67, (256, 256, 256), 21, 65536, ln=True), name="act8 control b65536"),
        # the paper's actor (three hidden layers of 2048) for a handful of environments
        dict(_mlp("act", 8, 67, (2048, 2048, 2048), 21, 16), name="act8 fc2048 b16"),
        # a wide policy at a batch that fills the chip
        dict(_mlp("act", 8, 256, (1024, 1024, 1024), 64, 16384), name="act8 wide b16384"),
        # frames from a few hundred emulators, greedy actions
        dict(_frames("act", 8, 84, 4, 32, 512, 18, 256), name="act8 frames b256"),
        # the paper's actor at q = 16, one observation at a time
        dict(_mlp("act", 16, 67, (2048, 2048, 2048), 21, 1), name="act16 fc2048 b1"),
        # the wide policy in half precision
        dict(_mlp("act", 16, 256, (1024, 1024, 1024), 64, 16384), name="act16 wide b16384"),
        # evaluation of the learner's own fp32 policy, at sizes that are no multiples of anything
        dict(_mlp("act", 32, 111, (400, 300), 8, 3001, ln=True), name="act32 control b3001"),
        # the learner's calibration of a frame policy: new parameters, ranges over a batch from replay
        dict(_frames("calibrate", 32, 84, 4, 32, 512, 18, 256), name="calibrate frames b256"),
        # one model pull of the paper's actor: quantize, hand over as a blob, install, act on it
        dict(_mlp("pull", 8, 67, (2048, 2048, 2048), 21, 16), name="pull fc2048"),
        # the quantizer on one weight tensor of 4 M values, for the broadcast
        {"do": "tensor", "rows": 2048, "cols": 2048, "scheme": "channel_sym_s8", "qdenom": 255, "name": "tensor 4M"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _batch(rng, hi, macs, most):
    """Log-uniform from 1, so that the case has at most `most` multiply-adds; half of the larger ones are whole tens."""
    b = _log(rng, 1, max(1, min(hi, most // macs)))
    return b if b < 100 or rng.random() < 0.5 else max(1, b // 16 * 16)


def draw(rng):
    do, bits = rng.choice([("act", 8)] * 8 + [("act", 16)] * 4 + [("act", 32)] * 2 + [("calibrate", 32)] * 2 +
                          [("pull", 8)] * 2 + [("tensor", 8)] * 2)
    if do == "tensor":
        cols = 4 * _log(rng, 8, 2048)
        rows = max(1, _log(rng, 1 << 16, 1 << 25) // cols)
        return {"do": do, "rows": rows, "cols": cols, "scheme": rng.choice(["channel_sym_s8", "tensor_asym_u8"]),
                "qdenom": rng.choice([255, 255, 255, 15])}
    most = {8: 39_000_000_000, 16: 39_000_000_000, 32: 2_300_000_000}[bits]
    if do != "pull" and rng.random() < 0.3:
        c = _frames(do, bits, rng.randint(52, 100), rng.choice([4, 4, 3, 1]), rng.choice([32, 32, 16]),
                    rng.choice([256, 512, rng.randint(100, 600)]), rng.randint(3, 18), 1)
        c["batch"] = _batch(rng, 2048, synth.macs_per_sample(_net(c)), most)
        return c
    # generic control policies: two or three hidden layers, equal or narrowing, round and odd widths
    kind = rng.random()
    if kind < 0.4:
        widths = (rng.choice([128, 256]),) * rng.choice([2, 3])
    elif kind < 0.6:
        widths = (rng.choice([512, 1024]),) * rng.choice([2, 3])
    elif kind < 0.75:
        widths = (2048,) * 3
    else:
        a = _log(rng, 48, 1100)
        widths = (a, rng.randint(max(32, a // 2), a))
    c = _mlp(do, bits, _log(rng, 8, 384), widths, rng.randint(1, 40), 1, ln=rng.random() < 0.4,
             scheme=rng.choice(["channel_sym_s8"] * 3 + ["tensor_asym_u8"]), explore=do == "act" and bits == 8 and rng.random() < 0.3,
             wbits=rng.choice([8, 8, 4]) if do == "pull" else 8)
    c["batch"] = _batch(rng, 65536 if do == "act" else 4096 if do == "calibrate" else 64, synth.macs_per_sample(_net(c)), most)
    return c


def _net(case):
    widths = [case[k] for k in ("width1", "width2", "width3") if case.get(k)]
    if case["net"] == "frames":
        h, c, layers = case["side"], case["stack"], []
        for out, k, stride in ((case["channels"], 8, 4), (2 * case["channels"], 4, 2), (2 * case["channels"], 3, 1)):
            layers.append(synth.conv(h, h, c, out, k, k, stride, "relu"))
            h, c = (h - k) // stride + 1, out
        k, in_type = h * h * c, "u8"
        head = "argmax" if case["bits"] == 8 else "linear"
    else:
        layers, k, in_type, head = [], case["inputs"], "f32", "tanh"
    for w in widths:
        layers.append(synth.fc(k, w, "ln_tanh" if case.get("ln") and not layers else "relu"))
        k = w
    layers.append(synth.fc(k, case["actions"], "none"))
    return dict(synth.small_net(layers, head=head, wscheme=case["scheme"], in_type=in_type), wbits=case["wbits"])


def _params(net, g):
    """Weights as training starts from, or stays close to in scale; frames are consumed as raw codes, so the first
    layer of a frame policy carries the 1/255."""
    w, b, gamma, beta = [], [], [], []
    for i, l in enumerate(net["layers"]):
        shape = synth.layer_weight_shape(l)
        fan_in = math.prod(shape[1:])
        scale = math.sqrt(2.0 / fan_in) / (255.0 if i == 0 and net["in_type"] == "u8" else 1.0)
        w.append(torch.randn(shape, generator=g, device=DEV) * scale)
        b.append(torch.empty(shape[0], device=DEV).uniform_(-0.1, 0.1, generator=g))
        ln = l["act"] == "ln_tanh"
        gamma.append(torch.empty(shape[0], device=DEV).uniform_(0.8, 1.2, generator=g) if ln else None)
        beta.append(torch.empty(shape[0], device=DEV).uniform_(-0.1, 0.1, generator=g) if ln else None)
    return w, b, gamma, beta


def _observations(net, batch, g):
    """Standardised vectors, or frames: flat regions with edges, the same scene moving on through the stack."""
    if net["in_type"] == "f32":
        return torch.randn((batch,) + synth.obs_shape(net), generator=g, device=DEV)
    h, w, c = synth.obs_shape(net)
    coarse = torch.randint(0, 256, (batch, h // 6 + 2, w // 6 + 2), generator=g, device=DEV, dtype=torch.uint8)
    scene = coarse.repeat_interleave(6, 1).repeat_interleave(6, 2)
    return torch.stack([scene[:, i:i + h, i:i + w] for i in range(c)], dim=3).contiguous()


def _ranges(net, params, obs):
    """Range of each layer's input over `obs` in plain fp32, outside the library: every build gets the same ones."""
    x = obs.float()
    out = []
    w, b, gamma, beta = params
    for i, l in enumerate(net["layers"]):
        lo, hi = torch.aminmax(x)
        out.append((float("%.3g" % min(0.0, float(lo))), float("%.3g" % max(0.0, float(hi)))))
        if l["kind"] == "conv":
            p = x.unfold(1, l["kh"], l["stride"]).unfold(2, l["kw"], l["stride"])  # [n, oh, ow, c, kh, kw]
            n, oh, ow = p.shape[:3]
            p = p.permute(0, 1, 2, 4, 5, 3).reshape(n * oh * ow, -1).contiguous()
            x = (p @ w[i].reshape(l["out_c"], -1).t().contiguous() + b[i]).reshape(n, oh, ow, l["out_c"])
        else:
            x = x.reshape(x.shape[0], -1) @ w[i].t().contiguous() + b[i]
        if l["act"] == "ln_tanh":
            x = torch.tanh(torch.nn.functional.layer_norm(x, x.shape[1:], gamma[i], beta[i], net["ln_eps"]))
        elif l["act"] == "relu":
            x = torch.relu(x)
    return out


def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    if case["do"] == "tensor":
        n = case["rows"] * case["cols"]
        rows = case["rows"] if case["scheme"] == "channel_sym_s8" else 1
        return {"case": case, "w": torch.randn((case["rows"], case["cols"]), generator=g, device=DEV) * 0.05,
                "codes": torch.empty(n, dtype=torch.uint8, device=DEV), "scale": torch.empty(rows, device=DEV),
                "zp": torch.empty(rows, dtype=torch.int32, device=DEV), "ws": torch.zeros(4096, dtype=torch.int32, device=DEV)}
    net, batch = _net(case), case["batch"]
    params = _params(net, g)
    obs = _observations(net, batch, g)
    s = {"case": case, "params": params, "obs": obs, "policy": aq.Policy(net)}
    if net["head"] == "argmax":
        s["actions"] = torch.zeros(batch, dtype=torch.int32, device=DEV)
    else:
        s["actions"] = torch.zeros((batch, case["actions"]), device=DEV)
    if case["bits"] == 8:
        rows = CALIBRATION_FRAMES if net["in_type"] == "u8" else CALIBRATION_ROWS
        s["ranges"] = _ranges(net, params, _observations(net, rows, g))
        s["sigma"] = torch.empty(batch, device=DEV).uniform_(0.0, 0.2, generator=g)
        s["seed"] = seed
    p = s["policy"]
    if case["do"] == "pull":
        s["actor"] = aq.Policy(net)
        size = p.policy_blob_size() if case["wbits"] == 8 else p.policy_packed_blob_size()
        s["blob"] = torch.zeros(size, dtype=torch.uint8, device=DEV)
        s["actor"].policy_reserve(batch)
    elif case["bits"] == 8:
        p.quantize_params(*params, s["ranges"])
        if p.policy_status() != aq.OK:
            raise RuntimeError("the policy could not be quantized")
    elif case["bits"] == 16:
        p.convert_params_fp16(*params)
    else:
        p.policy_set_params_fp32(*params)
    p.policy_reserve(batch)
    return s


def run(s):
    case = s["case"]
    if case["do"] == "tensor":
        rows, cols = case["rows"], case["cols"]
        if case["scheme"] == "tensor_asym_u8":
            rows, cols = 1, rows * cols
        aq.quantize_tensor(s["w"], rows, cols, case["scheme"], case["qdenom"], s["codes"], s["scale"], s["zp"], s["ws"])
        return {"codes": s["codes"], "scale": s["scale"], "zp": s["zp"]}
    p = s["policy"]
    if case["do"] == "calibrate":
        p.policy_set_params_fp32(*s["params"])
        return p.calibrate_fp32(s["obs"])
    if case["do"] == "pull":
        a = s["actor"]
        p.quantize_params(*s["params"], s["ranges"])
        if case["wbits"] == 8:
            p.policy_export_blob(s["blob"])
            a.policy_import_blob(s["blob"])
        else:
            p.policy_export_packed_blob(s["blob"])
            a.policy_import_packed_blob(s["blob"])
        a.policy_forward_int8(s["obs"], s["actions"])
        return {"blob": s["blob"], "actions": s["actions"]}
    if case["bits"] == 16:
        p.policy_forward_fp16(s["obs"], s["actions"])
    elif case["bits"] == 32:
        p.policy_forward_fp32(s["obs"], s["actions"])
    elif case["explore"]:
        p.policy_step_int8(s["obs"], s["actions"], s["seed"], 1, sigma=s["sigma"])
    else:
        p.policy_forward_int8(s["obs"], s["actions"])
    return s["actions"]


def work(case):
    if case["do"] == "tensor":
        n = case["rows"] * case["cols"]
        return {"bytes": 5 * n + (8 * case["rows"] if case["scheme"] == "channel_sym_s8" else 8), "flops": 0}
    net, batch = _net(case), case["batch"]
    weights = sum(math.prod(synth.layer_weight_shape(l)) for l in net["layers"])
    obs = batch * math.prod(synth.obs_shape(net)) * (1 if net["in_type"] == "u8" else 4)
    actions = batch * 4 * (1 if net["head"] == "argmax" else case["actions"])
    flops = 2 * synth.macs_per_sample(net) * batch
    if case["do"] == "pull":  # the fp32 parameters read, the blob written and read, the actor's weights read
        return {"bytes": 4 * weights + 3 * weights * case["wbits"] // 8 + obs + actions, "flops": flops}
    if case["do"] == "calibrate":  # the parameters read and kept, the observations read
        return {"bytes": 8 * weights + obs, "flops": flops - 2 * case["width1"] * case["actions"] * batch
                if case["net"] == "frames" else flops - 2 * net["layers"][-1]["in"] * case["actions"] * batch}
    return {"bytes": weights * case["bits"] // 8 + obs + actions, "flops": flops}


def tolerance(case):
    if case["do"] == "tensor":
        return "exact"
    if case["bits"] == 32:
        return {"rel": 1e-5}
    if case["bits"] == 16:
        return {"rel": 2e-3}  # every tensor is rounded to 11 bits: another order of the sums moves single values by one
    if case["net"] == "frames":
        return "exact"
    # whole numbers up to the head; behind a LayerNorm, whose statistics are fp32, single codes may round the other way
    return {"rel": 1e-3} if case["ln"] else {"rel": 1e-5}
