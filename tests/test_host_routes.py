"""Host code of the library on a HIP runtime of host memory (fake_hip.c): which kernels a forward launches on which stream and
buffers, what it allocates, and what it answers when a runtime call fails.  Each scenario runs in a process of its own, in
which no other HIP runtime is loaded."""
import ctypes as C
import itertools
import os
import re
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LAUNCH, MALLOC, WAIT, RECORD = range(4)


class Entry(C.Structure):
    _fields_ = [("kind", C.c_int), ("grid", C.c_uint * 3), ("stream", C.c_void_p), ("in_", C.c_void_p), ("out", C.c_void_p),
                ("flags", C.c_int), ("name", C.c_char * 160)]


class Mem:
    """What the binding asks of a tensor."""

    def __init__(self, rows=1):
        self._buf = C.create_string_buffer(4096)
        self.shape = (rows,)

    def data_ptr(self):
        return (C.addressof(self._buf) + 255) & ~255


class Host:
    def __init__(self, fake_path):
        sys.path.insert(0, ROOT)
        self.hip = C.CDLL(fake_path, mode=C.RTLD_GLOBAL)
        self.hip.fake_entry.restype = C.POINTER(Entry)
        for f in ("fake_capture", "fake_set_busy"):
            getattr(self.hip, f).argtypes = [C.c_void_p]
        from paper_1910_01055_amd import binding, synth
        self.aq, self.synth = binding, synth
        binding._stream = lambda: self.stream
        self.stream = 0

    def policy(self, *widths, k=67, out=21, wbits=0, ln=(), **kw):
        fc, layers = self.synth.fc, []
        for i, w in enumerate(widths):
            layers.append(fc(k, w, "ln_tanh" if i in ln else "relu"))
            k = w
        net = dict(self.synth.small_net(layers + [fc(k, out, "none")], **kw), wbits=wbits)
        P = self.aq.Policy(net)
        n = len(net["layers"])
        lns = [Mem() if i in ln else None for i in range(n)]
        P.quantize_params([Mem()] * n, [Mem()] * n, lns, lns, [(0.0, 1.0)] * n)
        return P

    def logged(self, kind=None):
        e = [self.hip.fake_entry(i).contents for i in range(self.hip.fake_entries())]
        return [x for x in e if kind is None or x.kind == kind]

    def forward(self, P, batch, stream=0):
        """-> the entries of one forward on `stream`."""
        self.stream = stream
        self.hip.fake_clear()
        P.policy_forward_int8(Mem(batch), Mem(batch))
        return self.logged()

    def maps(self, entries):
        """Addresses of the maps between the layers of a few-row forward; empty for one whole-network launch."""
        runs = [e for e in entries if e.kind == LAUNCH]
        if len(runs) == 1:
            assert b"mlp" in runs[0].name
            return set()
        assert all(b"k_layer_skinny" in e.name for e in runs)
        for a, b in zip(runs, runs[1:]):
            assert a.out == b.in_
        return {e.out for e in runs[:-1]}


def few_row_forwards_allocate_nothing(h):
    """... with or without a reserve, on any stream: a wide policy at few rows needed no memory on the whole-network kernels."""
    for reserve in (True, False):
        P = h.policy(1024, 1024)
        if reserve:
            P.policy_reserve(64)
        seen = []
        for stream in (0, 64, 128, 192, 320, 0):
            entries = h.forward(P, 16, stream)
            assert not [e for e in entries if e.kind == MALLOC], (reserve, stream)
            seen.append(h.maps(entries))
        assert len(seen[0]) == 2 and seen[5] == seen[0]
        assert len({m for s in seen[:4] for m in s}) == 8
        P.close()
    assert h.hip.fake_live() == 0


def policies_that_never_take_few_rows_apart_keep_no_maps(h):
    """One allocation for a policy, two where few rows run layer by layer."""
    for widths, n in (((256, 256), 1), ((300, 280), 1), ((1024, 1024), 2), ((2048, 2048), 1)):
        h.hip.fake_clear()
        P = h.policy(*widths)
        assert len(h.logged(MALLOC)) == n, widths
        assert (P.policy_fused_plan(1)[0] == 0) == (n == 2 or widths[0] == 2048)
        P.close()


def streams_come_and_go(h):
    """Pairs of maps are given back by streams that are done, and only by those; the default stream keeps its own without an
    event; a handle that names a new stream waits for what the old one left in flight."""
    P = h.policy(1024, 1024)
    default = h.maps(h.forward(P, 16))
    assert [e.kind for e in h.logged()] == [LAUNCH] * 3
    used = set(default)
    for n in range(1, 4):  # three streams at once, their work in flight
        h.hip.fake_set_busy(64 * n)
        entries = h.forward(P, 16, 64 * n)
        assert [e.kind for e in entries] == [LAUNCH] * 3 + [RECORD] and {e.stream for e in entries} == {64 * n}
        assert len(h.maps(entries)) == 2 and not used & h.maps(entries)
        used |= h.maps(entries)
    assert not h.maps(h.forward(P, 16, 1000))  # a fourth: the whole network in one launch
    mine = h.forward(P, 16, 128)  # a handle seen before, of a new stream perhaps
    assert [e.kind for e in mine] == [WAIT] + [LAUNCH] * 3 + [RECORD] and mine[0].in_ == mine[-1].in_
    h.hip.fake_finish_all()
    for n in range(20):  # a stream per episode
        entries = h.forward(P, 16, 2000 + 64 * n)
        assert len(h.maps(entries)) == 2 and not h.maps(entries) & default and entries[-1].kind == RECORD
    assert h.maps(h.forward(P, 16)) == default
    # the handle of each thread's own default stream is one like the others; a captured stream takes one launch
    assert len(h.maps(h.forward(P, 16, 2))) == 2
    h.hip.fake_capture(64)
    assert not h.maps(h.forward(P, 16, 64))
    P.close()
    assert h.hip.fake_live() == 0
    # where the event costs what the layers' launches gain
    Q = h.policy(512, 512)
    h.forward(Q, 16)
    assert h.maps(h.forward(Q, 16)) and not h.maps(h.forward(Q, 16, 128))


def the_first_forward_of_new_weights(h):
    """One launch where the layers' gain is what their round trips for cold weights cost; layers of 1024 gain more."""
    for widths, first in (((512, 512), False), ((1024, 1024), True)):
        P = h.policy(*widths)
        for renew in (lambda: None, lambda: P.quantize_params([Mem()] * 3, [Mem()] * 3, None, None, [(0.0, 1.0)] * 3)):
            renew()
            assert [bool(h.maps(h.forward(P, 16))) for _ in range(3)] == [first, True, True], widths
        P.close()


def fp32_convolutions_of_small_frames(h):
    """One launch for the convolutions while that is faster: not for rounds of images without number, each of which gives a CU one
    small frame."""
    conv, fc = h.synth.conv, h.synth.fc
    for side, stack, ch, one, many in ((84, 4, 32, (64, 256, 257, 300, 1000, 2048), ()), (52, 1, 16, (49, 256, 512), (1300, 2048, 4096)),
                                       (61, 3, 16, (100, 256, 512), (900, 1500, 2048)), (52, 3, 32, (100, 256, 512), (1300, 3000, 4096))):
        layers, n, c = [], side, stack
        for out, k, s in ((ch, 8, 4), (2 * ch, 4, 2), (2 * ch, 3, 1)):
            layers.append(conv(n, n, c, out, k, k, s, "relu"))
            n, c = (n - k) // s + 1, out
        net = h.synth.small_net(layers + [fc(n * n * c, 256, "relu"), fc(256, 6, "none")], head="linear", in_type="u8")
        P = h.aq.Policy(net)
        P.policy_set_params_fp32([Mem()] * 5, [Mem()] * 5, None, None)
        for batch in one + many:
            P.policy_reserve(batch)
            assert (P.policy_fp32_plan(batch)[1][0][0] == 0) == (batch in one), (side, stack, ch, batch)
            h.hip.fake_clear()
            P.policy_forward_fp32(Mem(batch), Mem(batch))
            names = [e.name for e in h.logged(LAUNCH)]
            assert len(names) == (3 if batch in one else 5) and any(b"conv_stack" in x for x in names) == (batch in one)
        P.close()


def half_precision_layers_by_their_output_tiles(h):
    """The last batch of the few-row kernel and the first of the tiled one, for each side of the rule: short and long K, few and many
    features, rows of whole 8 values and not, fp32 and 16-bit inputs.  (A layer of 6000 keeps the policy from one launch.)"""
    fc = h.synth.fc
    for layers, at, last in (([fc(16, 6000, "relu"), fc(6000, 128, "relu"), fc(128, 9, "none")], 1, 7968),
                             ([fc(16, 6000, "relu"), fc(6000, 128, "relu"), fc(128, 9, "none")], 2, 15968),
                             ([fc(16, 6000, "relu"), fc(6000, 200, "relu"), fc(200, 9, "none")], 2, 67168),
                             ([fc(16, 6000, "relu"), fc(6000, 200, "relu"), fc(200, 300, "relu"), fc(300, 9, "none")], 2, 4256),
                             ([fc(16, 6000, "relu"), fc(6000, 200, "relu"), fc(200, 128, "relu"), fc(128, 9, "none")], 2, 3968),
                             ([fc(16, 6001, "relu"), fc(6001, 128, "relu"), fc(128, 9, "none")], 1, 19968),
                             ([fc(16, 6000, "relu"), fc(6000, 100, "relu"), fc(100, 40, "none")], 2, 11168),
                             ([fc(200, 6000, "relu"), fc(6000, 9, "none")], 0, 256),
                             ([fc(203, 6000, "relu"), fc(6000, 9, "none")], 0, 320),
                             ([fc(16, 9, "relu"), fc(9, 6000, "relu"), fc(6000, 9, "none")], 0, 67168)):
        net = h.synth.small_net(layers, head="linear")
        P, n = h.aq.Policy(net), len(layers)
        P.convert_params_fp16([Mem()] * n, [Mem()] * n, None, None)
        for batch in (last, last + 1):
            P.policy_reserve(batch)
            h.hip.fake_clear()
            P.policy_forward_fp16(Mem(batch), Mem(batch))
            names = [e.name for e in h.logged(LAUNCH)]
            assert len(names) == n and (b"k_layer_fp16_rows" in names[at]) == (batch == last), (layers, batch, names)
        P.close()


def a_few_row_forward_without_memory_to_have(h):
    """... answers OK: it needs none."""
    P = h.policy(1024, 1024)
    h.hip.fake_fail_mallocs(1)
    assert len(h.maps(h.forward(P, 16, 64))) == 2


def a_failed_call_leaves_no_error_behind(h):
    """What the caller was told once is not told again by the next call, which works."""
    aq, hip = h.aq, h.hip

    def fails(status, f, *args):
        hip.fake_fail_mallocs(1)
        with pytest.raises(aq.AqError) as e:
            f(*args)
        assert e.value.status == status
        hip.fake_fail_mallocs(0)

    fails(aq.ENOMEM, h.policy, 1024, 1024)
    assert hip.fake_live() == 0
    P = h.policy(2048, 2048, wbits=4)  # a launch per layer: the forward needs memory
    P.policy_reserve(4)
    obs, out, pars = Mem(64), Mem(64), ([Mem()] * 3, [Mem()] * 3, None, None)
    for f, args in ((P.policy_reserve, (64,)), (P.policy_forward_int8, (obs, out)), (P.policy_set_path, (4,)), (P.convert_params_fp16, pars),
                    (P.policy_set_params_fp32, pars), (P.policy_forward_fp32_params, pars + (obs, out))):
        fails(aq.ENOMEM, f, *args)
        P.policy_forward_int8(Mem(4), Mem(4))
    P.policy_set_params_fp32(*pars)
    fails(aq.ENOMEM, P.calibrate_fp32, Mem(4))
    P.policy_forward_int8(Mem(4), Mem(4))
    # a stream that cannot be asked whether it is being captured: the whole network in one launch, and done
    Q = h.policy(1024, 1024)
    hip.fake_fail_capture_query(1)
    assert not h.maps(h.forward(Q, 16, 64)) and len(h.logged(LAUNCH)) == 1
    hip.fake_fail_capture_query(0)


def a_refused_amount_of_lds_is_told_once(h):
    """... by the call whose kernel asked for it; the same call later, where it is granted, works."""
    fc, conv, small = h.synth.fc, h.synth.conv, h.synth.small_net
    frames = small([conv(84, 84, 4, 32, 8, 8, 4, "relu"), conv(20, 20, 32, 64, 4, 4, 2, "relu"), conv(9, 9, 64, 64, 3, 3, 1, "relu"),
                    fc(3136, 512, "relu"), fc(512, 18, "none")], head="linear", in_type="u8")
    mlp = lambda *w: small([fc(a, b, "relu") for a, b in zip(w, w[1:])] + [fc(w[-1], 21, "none")])
    for net, batch, bits, kernel in ((mlp(67, 400, 300), 4096, 8, b"k_mlp_fused"), (mlp(256, 1024, 1024), 16384, 8, b"k_mlp_wide"),
                                     (mlp(67, 2048, 2048), 16384, 8, b"k_layer_int8"), (frames, 256, 8, b"k_conv_stack"),
                                     (mlp(67, 256), 4096, 16, b"k_fp16_mlp"), (frames, 256, 16, b"k_fp16_conv_stack"),
                                     (mlp(67, 256), 4096, 32, b"k_fp32_mlp"), (mlp(67, 2048), 4096, 32, b"k_fp32_layer"),
                                     (frames, 256, 32, b"k_fp32_conv_stack")):
        P, n = h.aq.Policy(net), len(net["layers"])
        P.quantize_params([Mem()] * n, [Mem()] * n, None, None, [(0.0, 1.0)] * n)
        P.convert_params_fp16([Mem()] * n, [Mem()] * n, None, None)
        P.policy_set_params_fp32([Mem()] * n, [Mem()] * n, None, None)
        P.policy_reserve(batch)
        call = {8: P.policy_forward_int8, 16: P.policy_forward_fp16, 32: P.policy_forward_fp32}[bits]
        h.hip.fake_fail_attributes(1)
        with pytest.raises(h.aq.AqError) as e:
            call(Mem(batch), Mem(batch))
        assert e.value.status == h.aq.EHIP
        h.hip.fake_fail_attributes(0)
        h.hip.fake_clear()
        call(Mem(batch), Mem(batch))
        assert any(kernel in x.name for x in h.logged(LAUNCH)), (kernel, [x.name for x in h.logged(LAUNCH)])
        P.close()


def layer_launch(e):
    """-> (kernel, how it reads its input, how it leaves its output); "own" is an order nobody else reads or writes."""
    name, flags = e.name.decode(), e.flags
    if "k_layer_rows" in name:
        return "rows", "own" if "k_layer_rowsILb1E" in name else "operands", "own" if flags & 2 else "operands"
    if "k_layer_skinny" in name:
        reads = ("own", "rows", "operands")[int(re.search(r"Li(\d)EEEv", name).group(1))]
        return "skinny", reads, "own" if flags & (2 | 4) else "operands" if flags & 64 else "rows"
    if "k_layer_int8" in name:
        assert not flags, "the tiled kernel knows row-major maps only"
        return "tiled", "rows", "rows"
    if "k_ln_tanh" in name:
        return "ln", "own", "operands" if flags else "rows"
    return name, "own", "own"


WIDE = {  # hidden widths, outputs, layers with a LayerNorm
    "2048x3": ((2048, 2048, 2048), 21, ()), "2048x3 ln": ((2048, 2048, 2048), 21, (0,)), "2048x2-256": ((2048, 2048, 256), 21, ()),
    "2048x2-256 ln": ((2048, 2048, 256), 21, (0, 1)), "1300x2-400": ((1300, 1300, 400), 21, ()), "1300x2-400 ln": ((1300, 1300, 400), 21, (2,)),
    "2048x2, wide last": ((2048, 2048), 512, ()), "2048x2, wide last ln": ((2048, 2048), 512, (1,)), "1100-700": ((1100, 700), 21, ()),
    "1100-200-1030": ((1100, 200, 1030), 21, ()), "1100-200-1030 ln": ((1100, 200, 1030), 21, (0, 2)), "200-1300-1300": ((200, 1300, 1300), 21, ()),
    "1100-1000-1030-30": ((1100, 1000, 1030, 30), 5, (1, 3)), "1300": ((1300,), 300, ()),
    "1024x2-300": ((1024, 1024, 300), 9, (1,)), "800-600": ((800, 600), 9, ())}
WIDE_BATCHES = (1, 449, 450, 640, 900, 960, 961, 1300, 3000, 4500, 8000, 8128, 8129, 8150, 8191, 8192, 9000)


def wide_layers_read_the_order_their_input_was_written_in(h):
    """A kernel that writes operand order is only followed by one that reads it, for every mixture of widths, on both sides of where
    each of the three kernels begins and ends, from every entry point; narrower policies, too, where a plan makes them go by layers."""
    seen = set()

    def static(P, batch):
        h.hip.fake_clear()
        try:
            P.policy_forward_int8_static(Mem(batch), Mem(batch))
        except h.aq.AqError as e:
            assert e.status == h.aq.ETOOBIG
        return h.logged()

    def step(P, batch):
        h.hip.fake_clear()
        P.policy_step_int8(Mem(batch), Mem(batch), 1, 1, sigma=Mem(batch))
        return h.logged()

    for name, (widths, out, ln) in WIDE.items():
        for scheme, head in itertools.product(("channel_sym_s8", "tensor_asym_u8"), ("linear", "argmax")):
            P = h.policy(*widths, out=out, ln=ln, wscheme=scheme, head=head)
            P.policy_set_path(2)
            for batch in WIDE_BATCHES:
                for call in (h.forward, static, step)[:2 if head == "argmax" else 3]:
                    case, runs = (name, scheme, head, batch), [layer_launch(e) for e in call(P, batch) if e.kind == LAUNCH]
                    assert not runs or sum(r[0] in ("rows", "skinny", "tiled") for r in runs) == len(widths) + 1, (case, runs)
                    order = None  # of the last map written
                    for kernel, reads, writes in runs:
                        if order is not None and kernel in ("rows", "skinny", "tiled"):
                            assert reads == order, (case, runs)
                        if kernel in ("rows", "skinny", "tiled", "ln"):
                            order = writes if writes != "own" else order
                    seen.update((name, batch, r[0]) for r in runs)
            P.close()
    # where the many-row kernel serves and where it does not, because its reader could not follow
    for name, batch, many in (("2048x3", 449, False), ("2048x3", 450, True), ("2048x3", 8128, True), ("2048x3", 8129, False),
                              ("2048x2-256", 1300, True), ("2048x2-256 ln", 1300, True), ("1300x2-400", 3000, True), ("2048x2, wide last", 4500, False),
                              ("1100-200-1030", 450, False), ("1100-200-1030", 900, True), ("200-1300-1300", 640, False), ("200-1300-1300", 900, True), ("1300", 900, True)):
        assert ((name, batch, "rows") in seen) == many, (name, batch)


def wide_layers_behind_the_first_at_some_hundred_rows(h):
    """They go to the many-row kernel where its grid holds enough workgroups, or their rows are long, else to the few-row one."""
    sym, asym = "channel_sym_s8", "tensor_asym_u8"
    for widths, scheme, at in (((2048,) * 3, sym, 769), ((2048,) * 3, asym, 897), ((1100,) * 3, sym, 1025), ((1100,) * 3, asym, 1281),
                               ((1100, 700), sym, 1537), ((1100, 512), sym, 2177), ((2500,) * 2, sym, 450), ((2500,) * 2, asym, 450)):
        P = h.policy(*widths, wscheme=scheme)
        for batch in (max(at - 1, 450), at):
            want = ["rows"] + ["rows" if batch >= at else "skinny"] * (len(widths) - 1) + ["skinny"]
            assert [layer_launch(e)[0] for e in h.forward(P, batch) if e.kind == LAUNCH] == want, (widths, scheme, batch)
        P.close()
    # the first one stays on the few-row kernel while that takes tiles of 16 rows; one behind a few-row layer needs no other
    for widths, batch, want in (((1100, 300), 450, ["skinny"] * 3), ((1100, 300), 500, ["rows", "skinny", "skinny"]),
                                ((300, 1300, 1300), 1200, ["skinny", "rows", "rows", "skinny"]), ((1100, 700, 1100), 1200, ["rows", "skinny", "rows", "skinny"])):
        P = h.policy(*widths)
        assert [layer_launch(e)[0] for e in h.forward(P, batch) if e.kind == LAUNCH] == want, (widths, batch)
        P.close()


def long_layernorm_rows_without_number(h):
    """Rows of more than 1024 values: four wavefronts each as long as a launch holds so many, then the kernel of one wavefront a row, which
    takes four times as many rows."""
    fc = h.synth.fc
    net = h.synth.small_net([fc(37, 1100, "ln_tanh"), fc(1100, 1300, "relu"), fc(1300, 5, "none")])  # (too wide for one launch)
    P, ln = h.aq.Policy(net), [Mem(), None, None]
    P.quantize_params([Mem()] * 3, [Mem()] * 3, ln, ln, [(0.0, 1.0)] * 3)
    P.convert_params_fp16([Mem()] * 3, [Mem()] * 3, ln, ln)
    P.policy_set_params_fp32([Mem()] * 3, [Mem()] * 3, ln, ln)
    for forward, name in ((P.policy_forward_int8, b"k_ln_tanh"), (P.policy_forward_fp16, b"k_fp16_ln_tanh"), (P.policy_forward_fp32, b"k_fp32_ln_tanh")):
        for batch in ((1 << 24) - 1, 1 << 24, (1 << 26) - 4):
            h.hip.fake_clear()
            forward(Mem(batch), Mem(batch))
            names = [e.name for e in h.logged(LAUNCH) if name in e.name]
            assert len(names) == 1 and (b"_long" in names[0]) == (batch >= 1 << 24), (batch, names)
    P.close()


def rows_per_workgroup_of_the_general_kernel(h):
    """Whole rounds of two workgroups of 32 rows per CU are never given up for 64 rows; behind them only large policies take 64."""
    sym, asym = "channel_sym_s8", "tensor_asym_u8"
    for widths, ln, scheme, want in (((512, 256), (), sym, 32), ((512, 512), (), sym, 64), ((512, 400), (), sym, 32), ((512,) * 3, (), sym, 64), ((512,) * 3, (0,), sym, 32),
                                     ((512,) * 3, (), asym, 32), ((480,) * 3, (), sym, 32), ((490,) * 3, (), sym, 64)):
        P = h.policy(*widths, ln=ln, wscheme=scheme)
        rows = {b: P.policy_fused_plan(b)[0] for b in (4096, 4097, 16353, 16384, 16385, 24576, 24577)}
        assert rows == {4096: 16, 4097: 32, 16353: 32, 16384: 32, 16385: want, 24576: want,
                        24577: 128 if scheme == sym else 64}, (widths, ln, scheme, rows)
        P.close()


SCENARIOS = [rows_per_workgroup_of_the_general_kernel, long_layernorm_rows_without_number, wide_layers_behind_the_first_at_some_hundred_rows, wide_layers_read_the_order_their_input_was_written_in, few_row_forwards_allocate_nothing, streams_come_and_go, the_first_forward_of_new_weights, fp32_convolutions_of_small_frames, half_precision_layers_by_their_output_tiles, policies_that_never_take_few_rows_apart_keep_no_maps,
             a_few_row_forward_without_memory_to_have, a_failed_call_leaves_no_error_behind, a_refused_amount_of_lds_is_told_once]


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("hip") / "libamdhip64.so.7")
    subprocess.run(["gcc", "-O1", "-std=c11", "-Wall", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7", "-o", lib,
                    os.path.join(HERE, "fake_hip.c")], check=True)
    return lib


@pytest.mark.parametrize("name", [s.__name__ for s in SCENARIOS])
def test_host(fake, name):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), fake, name], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    {s.__name__: s for s in SCENARIOS}[sys.argv[2]](Host(sys.argv[1]))
