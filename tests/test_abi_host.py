"""CPU-only checks of the C-ABI library: it loads, exports every declared symbol, and rejects bad arguments on the
host before anything is launched (no GPU is touched by these calls)."""
import ctypes as C
import os
import re

import pytest
import torch

from paper_2511_15927_amd import binding as bd
from paper_2511_15927_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "bimamba.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(bimamba_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = declared_functions()
    assert set(names) == set(bd.EXPORTS)
    lib = bd.lib()
    for n in names:
        assert hasattr(lib, n), n
    assert bd.bimamba_version() == 1


def good():
    cfg = synth.mixer_cfg(2, 64, 128, io="bf16")
    desc = bd.make_desc(cfg)
    fake = 0x1000
    p = bd.Params(fake, fake, fake, fake, None)
    t = lambda ch: bd.Tensor(fake, 64 * ch, ch)
    inp = bd.Inputs(t(128), t(128), t(128), t(16), t(16))
    return cfg, desc, p, inp, t(128)


def call_fwd(desc, pf, pb, inp, out, ws=0x1000, ws_bytes=1 << 40):
    return bd.lib().bimamba_fwd(C.byref(desc), C.byref(pf) if pf else None, C.byref(pb) if pb else None,
                                C.byref(inp) if inp else None, None, C.byref(out) if out else None,
                                C.c_void_p(ws), ws_bytes, None)


def test_null_and_shape_errors_are_decided_on_the_host():
    cfg, desc, p, inp, out = good()
    assert call_fwd(desc, None, p, inp, out) == -1
    assert call_fwd(desc, p, p, None, out) == -1
    assert call_fwd(desc, p, p, inp, None) == -1
    assert call_fwd(desc, bd.Params(None, None, 0x1000, 0x1000, None), p, inp, out) == -1
    assert call_fwd(desc, p, p, inp, out, ws=None) == -1
    assert call_fwd(desc, p, p, inp, out, ws_bytes=16) == -5
    assert call_fwd(desc, p, p, inp, out, ws=0x1004) == -4
    bad = bd.Inputs(bd.Tensor(0x1001, 64 * 128, 128), inp.z, inp.dt, inp.B, inp.C)
    assert call_fwd(desc, p, p, bad, out) == -4
    narrow = bd.Inputs(bd.Tensor(0x1000, 64 * 128, 100), inp.z, inp.dt, inp.B, inp.C)
    assert call_fwd(desc, p, p, narrow, out) == -2
    overlap = bd.Inputs(bd.Tensor(0x1000, 128, 128), inp.z, inp.dt, inp.B, inp.C)
    assert call_fwd(desc, p, p, overlap, out) == -2
    wide = bd.Inputs(bd.Tensor(0x1000, 64 * ((1 << 26) + 1), (1 << 26) + 1), inp.z, inp.dt, inp.B, inp.C)
    assert call_fwd(desc, p, p, wide, out) == -3                 # token stride beyond what a tile's 32-bit row offsets reach


def call_bwd(desc, pf, pb, inp, inp_b, dout, gi, gi_b, qf, qb, ws=0x1000, ws_bytes=1 << 40):
    ref = lambda v: C.byref(v) if v is not None else None
    return bd.lib().bimamba_bwd(C.byref(desc), ref(pf), ref(pb), ref(inp), ref(inp_b), ref(dout), ref(gi), ref(gi_b),
                                ref(qf), ref(qb), C.c_void_p(ws), ws_bytes, None)


def test_gradient_call_errors_are_decided_on_the_host():
    cfg, desc, p, inp, dout = good()
    t = lambda ch, at=0x1000: bd.Tensor(at, 64 * ch, ch)
    gi, gi2 = bd.InputGrads(t(128), t(128), t(128), 0x1000, 0x1000), bd.InputGrads(t(128), t(128), t(128), 0x1000, 0x1000)
    qf, qb = bd.ParamGrads(0x1000, None, 0x1000, 0x1000, None), bd.ParamGrads(0x1000, None, 0x1000, 0x1000, None)
    need = bd.bimamba_bwd_workspace_bytes(desc)
    assert need > 0
    assert call_bwd(desc, p, p, inp, None, dout, gi, None, qf, qb, ws_bytes=need - 1) == -5
    assert call_bwd(desc, p, p, inp, None, dout, gi, None, qf, qb, ws=None) == -1
    assert call_bwd(desc, p, p, inp, None, dout, gi, None, qf, qb, ws=0x1008) == -4
    assert call_bwd(desc, None, p, inp, None, dout, gi, None, qf, qb) == -1
    assert call_bwd(desc, p, p, None, None, dout, gi, None, qf, qb) == -1
    assert call_bwd(desc, p, p, inp, None, None, gi, None, qf, qb) == -1
    assert call_bwd(desc, p, p, inp, None, dout, None, None, qf, qb) == -1
    assert call_bwd(desc, p, p, inp, None, dout, gi, None, None, qb) == -1
    assert call_bwd(desc, p, p, inp, None, dout, gi, None, qf, qf) == -8        # the two directions' parameter gradients alias
    # shared activations take one set of input gradients, separate activations need two
    assert call_bwd(desc, p, p, inp, None, dout, gi, gi2, qf, qb) == -1
    other = bd.Inputs(t(128, 0x9000), inp.z, inp.dt, inp.B, inp.C)
    assert call_bwd(desc, p, p, inp, other, dout, gi, None, qf, qb) == -1
    no_db = bd.InputGrads(t(128), t(128), t(128), None, 0x1000)
    assert call_bwd(desc, p, p, inp, None, dout, no_db, None, qf, qb) == -1
    odd = bd.InputGrads(t(128), t(128), t(128), 0x1002, 0x1000)
    assert call_bwd(desc, p, p, inp, None, dout, odd, None, qf, qb) == -4
    narrow = bd.InputGrads(bd.Tensor(0x1000, 64 * 128, 100), t(128), t(128), 0x1000, 0x1000)
    assert call_bwd(desc, p, p, inp, None, dout, narrow, None, qf, qb) == -2
    assert call_bwd(desc, p, p, inp, None, dout, gi, None, bd.ParamGrads(None, None, 0x1000, 0x1000, None), qb) == -1
    # layouts the gradient kernels do not cover are refused, whatever else is passed
    m2 = bd.make_desc(synth.m2_cfg(2, 64, 128, headdim=64, d_state=64))
    assert call_bwd(m2, p, p, inp, None, dout, gi, None, qf, qb) == -3
    assert bd.bimamba_bwd_workspace_bytes(m2) == 0
    n32 = bd.make_desc(synth.mixer_cfg(2, 64, 128, d_state=32))
    assert call_bwd(n32, p, p, inp, None, dout, gi, None, qf, qb) == -3


@pytest.mark.parametrize("field,value,code", [
    ("struct_size", 8, -2), ("batch", -1, -2), ("seqlen", -5, -2), ("d_inner", 0, -2), ("n_heads", 3, -2),
    ("n_groups", 5, -2), ("d_state", 12, -3), ("d_conv", 5, -3), ("d_conv", 0, -2), ("io_dtype", 7, -3),
    ("a_kind", 2, -3), ("d_kind", 9, -3), ("combine", 2, -3), ("dt_softplus", 2, -3), ("conv_bc", -1, -3),
    ("time_chunks", -1, -2), ("state_split", -1, -2), ("state_split", 3, -3), ("state_split", 8, -3),
])
def test_descriptor_validation(field, value, code):
    cfg, desc, p, inp, out = good()
    setattr(desc, field, value)
    assert call_fwd(desc, p, p, inp, out) == code
    assert bd.bimamba_workspace_bytes(desc) == 0
    assert bd.bimamba_time_chunks(desc) == 0


def test_group_tiling_rule():
    cfg = synth.mixer_cfg(1, 8, 96, n_heads=96, n_groups=2)      # 48 channels per group: a wave would straddle groups
    desc = bd.make_desc(cfg)
    assert bd.bimamba_workspace_bytes(desc) == 0


def test_workspace_and_chunk_planning():
    d1 = bd.make_desc(synth.CONFIGS["headline"])
    assert bd.bimamba_time_chunks(d1) == 1                       # chains x 2 lanes per chain already fill the chip
    d2 = bd.make_desc(synth.CONFIGS["cfg2"])
    assert bd.bimamba_time_chunks(d2) == 128                     # batch 1: one lane per chain, 16 waves per SIMD from time segments
    assert bd.bimamba_time_chunks(bd.make_desc(synth.CONFIGS["cfg3_block"])) == 1
    assert bd.bimamba_time_chunks(bd.make_desc(synth.mixer_cfg(1, 100, 64, time_chunks=7))) == 7
    assert bd.bimamba_time_chunks(bd.make_desc(synth.mixer_cfg(1, 5, 64, time_chunks=7))) == 5
    assert bd.bimamba_time_chunks(bd.make_desc(synth.mixer_cfg(1, 256, 512))) == 1     # one launch, no segments across workgroups
    # (the one-launch form costs 4 states as much as 16, the segments do not: beyond 0.75 M channel tokens they are cut)
    short = {n: bd.bimamba_time_chunks(bd.make_desc(synth.mixer_cfg(2, 181, 2864, d_state=n))) for n in (4, 8, 16)}
    assert short[4] > 1 and short[8] == short[16] == 1, short
    # batch sweep at d_inner 4096 (w = 128 waves per batch element with one lane per chain): whole sequence with two
    # lanes per chain from 1.7 to 5 waves per SIMD (batch 7-20), with one lane per chain above, time segments below
    chunks = {b: bd.bimamba_time_chunks(bd.make_desc(synth.mixer_cfg(b, 8192, 4096))) for b in (1, 4, 6, 7, 8, 12, 16, 20, 21, 24, 64)}
    assert [b for b, n in chunks.items() if n == 1] == [7, 8, 12, 16, 20, 21, 24, 64], chunks
    assert chunks[1] == 32 and chunks[4] == 32 and chunks[6] > 1
    sep = bd.make_desc(synth.mixer_cfg(8, 8192, 4096, combine=1))
    assert bd.bimamba_workspace_bytes(sep) < bd.bimamba_workspace_bytes(d1)     # no partial buffer without ADD
    assert bd.bimamba_workspace_bytes(d1) % 256 == 0


@pytest.mark.parametrize("batch,L,Dn", [(4, 1931, 1600), (7, 635, 2944), (5, 4345, 512)])
def test_full_sequence_calls_are_not_planned_for_the_static_scratch(batch, L, Dn):
    """Calls whose segments by cost need a little more than the fixed scratch of the static block entry point: the block
    variant is held to segments that fit it, a full-sequence call is not.  Its segments are those of the same call without a
    partial buffer, which fits the scratch anyway."""
    add, sep = (bd.make_desc(synth.mixer_cfg(batch, L, Dn, combine=c)) for c in (0, 1))
    assert bd.bimamba_workspace_bytes(sep, 0) == bd.bimamba_workspace_bytes(sep, 1) < bd.STATIC_SCRATCH_BYTES
    assert bd.bimamba_workspace_bytes(add, 1) <= bd.STATIC_SCRATCH_BYTES < bd.bimamba_workspace_bytes(add, 0)
    assert bd.bimamba_time_chunks(add) == bd.bimamba_time_chunks(sep)


@pytest.mark.parametrize("N", [4, 8, 16])
@pytest.mark.parametrize("batch,L,Dn", [(1, 300, 64), (3, 600, 128), (1, 1928, 256), (2, 6000, 256), (1, 16384, 64), (1, 32768, 16)])
def test_narrow_sequences_are_cut_into_segments(batch, L, Dn, N):
    """Calls with too few chains to fill the chip, however short the segments: they are cut all the same, into segments of at
    least half the root of the sequence (the carry folds them one after the other), not walked whole."""
    n = bd.bimamba_time_chunks(bd.make_desc(synth.mixer_cfg(batch, L, Dn, d_state=N)))
    assert 8 <= n <= 2 * L ** 0.5, n
    assert 16 <= L // n


def test_time_parts_of_the_matrix_core_path():
    # 64 heads: batch 1 leaves 3/4 of the CUs empty -> 4 parts; batch 2 would have 2 and meets in the middle; batch 4 fills the chip -> 1.
    parts = {b: bd.bimamba_time_chunks(bd.make_desc(synth.m2_cfg(b, 8192, 4096))) for b in (1, 2, 3, 4, 8)}
    assert parts == {1: 4, 2: 1, 3: 1, 4: 1, 8: 1}, parts
    # directions kept apart share a launch anyway: twice the items, never met in the middle
    parts = {b: bd.bimamba_time_chunks(bd.make_desc(synth.m2_cfg(b, 8192, 4096, combine=1))) for b in (1, 2, 4)}
    assert parts == {1: 2, 2: 1, 4: 1}, parts
    # 8 heads: 16 parts at most, and no part shorter than 8 chunks of 64 tokens
    assert bd.bimamba_time_chunks(bd.make_desc(synth.m2_cfg(1, 32768, 512))) == 16
    assert bd.bimamba_time_chunks(bd.make_desc(synth.m2_cfg(1, 2048, 512))) == 4
    for L, apart in ((1023, 2), (960, 1), (17 * 64, 2)):     # parts of ceil(chunks / parts) chunks: 17 chunks in 2 parts of 9
        assert bd.bimamba_time_chunks(bd.make_desc(synth.m2_cfg(1, L, 512, combine=1))) == apart
        assert bd.bimamba_time_chunks(bd.make_desc(synth.m2_cfg(1, L, 512))) == 1     # (two parts at most: met in the middle)
    # the part states live in the workspace
    one = bd.bimamba_workspace_bytes(bd.make_desc(synth.m2_cfg(4, 8192, 4096))) / 4
    assert bd.bimamba_workspace_bytes(bd.make_desc(synth.m2_cfg(1, 8192, 4096))) > one
    # the block variant keeps one part (a block is at most a few chunks)
    assert bd.bimamba_time_chunks(bd.make_desc(synth.m2_cfg(1, 64, 512))) == 1


def test_output_overlapping_an_input_is_rejected_on_the_host():
    """out may not overlap any input view: same buffer in place, a partial overlap, or interleaved columns that collide.
    Column slices of one buffer that stay apart are legal (they are not reached here: a legal call would launch)."""
    cfg, desc, p, inp, out = good()
    Dn, L = 128, 64
    elem = 2
    base = 0x100000
    pitch = 4 * Dn                                                    # one projection buffer, row pitch 512 elements
    col = lambda c, ch: bd.Tensor(base + c * elem, L * pitch, pitch)
    sliced = bd.Inputs(col(0, Dn), col(Dn, Dn), col(2 * Dn, Dn), col(3 * Dn, 16), col(3 * Dn + 16, 16))
    assert call_fwd(desc, p, p, sliced, col(0, Dn)) == -8             # in place over x
    assert call_fwd(desc, p, p, sliced, col(Dn - 1, Dn)) == -8        # columns straddle x and z
    assert call_fwd(desc, p, p, sliced, col(3 * Dn + 8, Dn)) == -8    # wraps over B, C and into the next row's x
    assert call_fwd(desc, p, p, sliced, bd.Tensor(base + (2 * L - 1) * pitch * elem, L * Dn, Dn)) == -8
    # (a column slice of the same buffer that no input uses passes the check: the next error comes from the missing GPU
    # or, on the GPU machine, the call runs; the GPU tests cover that case)
    assert lib_status_alias() == "the output overlaps an input"


def lib_status_alias():
    return bd.lib().bimamba_status_string(-8).decode()


def test_status_strings():
    lib = bd.lib()
    for code in range(0, -9, -1):
        assert lib.bimamba_status_string(code).decode() not in ("", "unknown status")
    assert lib.bimamba_status_string(-99).decode() == "unknown status"


@pytest.mark.parametrize("kind", ["same", "strided", "other_dtype", "own", "grad"])
@pytest.mark.parametrize("at_once", [False, True])
def test_step_inputs_refreshed_together_or_one_by_one(kind, at_once, monkeypatch):
    """A step's tensors are refreshed in one go where they are of the buffer's kind, one by one otherwise and in host memory: the same
    values at odd sizes.  (One go: as on a GPU, the library's copy stood in for by one of its places in host memory.)"""
    from paper_2511_15927_amd.decode import BlockDecodeLoop
    cfg = synth.mixer_cfg(2, 3, 5, d_state=4)
    layer = (synth.make_params(cfg, 1, 0), synth.make_params(cfg, 1, 1))
    loop = BlockDecodeLoop(cfg, [layer], 2, device="cpu")
    want = {k: v.to(torch.bfloat16) for k, v in synth.make_inputs(cfg, 3).items()}
    statuses = []

    def copy(desc, src, dst, stream=None, check=True):
        flat = loop._step_flat[0]
        widths = dict(x=5, z=5, dt=5, B=4, C=4)
        inside = lambda p: flat.data_ptr() <= p < flat.data_ptr() + flat.numel() * 2
        statuses.append(-8 if any(inside(getattr(src, k).ptr) for k in widths) else 0)
        if statuses[-1] == 0:
            for k, n in widths.items():
                s, d = getattr(src, k), getattr(dst, k)
                for b in range(2):
                    for t in range(3):
                        C.memmove(d.ptr + 2 * (b * d.stride_batch + t * d.stride_token), s.ptr + 2 * (b * s.stride_batch + t * s.stride_token), 2 * n)
        return statuses[-1]
    if at_once:
        monkeypatch.setattr(bd, "bimamba_copy_inputs", copy)
        monkeypatch.setattr(torch.cuda, "current_device", lambda: -1)
        loop._copies_at_once = True
    given = dict(want)
    if kind == "strided":
        given["x"] = want["x"].transpose(0, 1).contiguous().transpose(0, 1)
    elif kind == "other_dtype":
        given["z"] = want["z"].float()
    elif kind == "own":
        loop.set_step_inputs(0, want)
        given = dict(loop.step_inputs[0])
    elif kind == "grad":
        given["dt"] = want["dt"].clone().requires_grad_()
    statuses.clear()
    version = loop._step_flat[0]._version
    with torch.no_grad():
        loop.set_step_inputs(0, given)
    for k, v in want.items():
        assert torch.equal(loop.step_inputs[0][k], v.reshape(loop.step_inputs[0][k].shape)), k
    assert all(t.count_nonzero() == 0 for t in loop.step_inputs[1].values())
    assert statuses == ([] if not at_once else {"same": [0], "strided": [0], "own": [-8]}.get(kind, []))
    assert loop._step_flat[0]._version > version


@pytest.mark.parametrize("replaced", [("x",), ("dt", "C"), ("x", "z", "dt", "B", "C")])
def test_step_inputs_go_to_the_tensors_that_stand_there(replaced):
    """step_inputs is the caller's to read and to fill: the calls take what stands in it, so that is what is written."""
    from paper_2511_15927_amd.decode import BlockDecodeLoop
    cfg = synth.mixer_cfg(2, 8, 12, d_state=4)
    loop = BlockDecodeLoop(cfg, [(synth.make_params(cfg, 1, 0), synth.make_params(cfg, 1, 1))], 2, device="cpu")
    for k in replaced:
        loop.step_inputs[0][k] = torch.zeros_like(loop.step_inputs[0][k])
    given = {k: v.to(torch.bfloat16) for k, v in synth.make_inputs(cfg, 3).items()}
    loop.set_step_inputs(0, given)
    for k, t in loop.step_inputs[0].items():
        assert torch.equal(t, given[k].reshape(t.shape)), k
    assert all(t.count_nonzero() == 0 for t in loop.step_inputs[1].values())


def test_stack_errors_are_decided_on_the_host():
    """bimamba_block_stack: 2 layers x 2 steps; every argument error, and outputs that overlap an input of any step (those that share
    a projection's rows with the inputs without overlapping pass the check and are not reached here: they would launch)."""
    L, Dn, N = 32, 64, 16
    desc = bd.make_desc(synth.mixer_cfg(1, L, Dn))
    at = lambda i: 0x100000 * (i + 1)      # nothing is read
    view = lambda p, ch, st=None: bd.Tensor(p, L * (st or ch), st or ch)
    params = bd.Params(at(0), at(0), at(0), at(0), None)
    layer = bd.StackLayer(params, params, at(1), at(2))
    step = lambda i: bd.Inputs(view(at(i), Dn), view(at(i + 1), Dn), view(at(i + 2), Dn), view(at(i + 3), N), view(at(i + 4), N))
    fake = lambda p: type("T", (), dict(data_ptr=lambda self: p))()

    def call(layers=(layer, layer), steps=(step(3), step(8)), outs=(None, None, None, at(20)), desc=desc, counts=(2, 2), host=True, dev=0x1000):
        table = C.create_string_buffer(bd.make_stack_table(layers, steps, [None if o is None else fake(o) for o in outs]))
        return bd.lib().bimamba_block_stack(C.byref(desc), *counts, C.addressof(table) if host is True else host, dev, None)

    assert call(host=None) == -1 and call(dev=None) == -1
    assert call(dev=0x1004) == -4
    assert call(counts=(-1, 2)) == -2 and call(counts=(2, -1)) == -2
    assert call(counts=(0, 2)) == 0 and call(counts=(2, 0)) == 0          # nothing to do
    for over in (dict(time_chunks=1), dict(state_split=1), dict(combine=1), dict(d_state=32), dict(conv_bc=1), dict(seqlen=257), dict(batch=0)):
        assert call(desc=bd.make_desc(synth.mixer_cfg(1, L, Dn), **over)) == -3, over
    no_a, odd_a = bd.Params(at(0), at(0), None, at(0), None), bd.Params(at(0), at(0), at(0) + 2, at(0), None)
    for bad, code in ((bd.StackLayer(params, no_a, at(1), at(2)), -1), (bd.StackLayer(odd_a, params, at(1), at(2)), -4),
                      (bd.StackLayer(params, params, at(1) + 2, at(2)), -4), (bd.StackLayer(params, params, at(1), at(2) + 1), -4)):
        assert call(layers=(layer, bad)) == code
    good_step = step(8)
    for field, bad, code in (("z", bd.Tensor(None, L * Dn, Dn), -1), ("dt", view(at(3) + 1, Dn), -4), ("B", view(at(3), N, N - 1), -2),
                             ("x", view(at(3), Dn, (1 << 26) + 1), -3)):
        other = bd.Inputs(*[bad if f == field else getattr(good_step, f) for f, _ in bd.Inputs._fields_])
        assert call(steps=(step(3), other)) == code, field
    assert call(outs=(None, at(20) + 1, None, at(21))) == -4
    assert call(outs=(at(3), None, None, at(20))) == -8                    # in place over the first step's x
    assert call(outs=(at(10) + 2 * Dn * (L - 1), None, None, at(20))) == -8   # the last row of the second step's dt, by a first-step output
    assert call(outs=(None, None, None, at(12) - 2 * Dn * L + 2)) == -8    # ends in the first value of the second step's C


def test_a_block_can_be_captured_without_a_run_before(monkeypatch):
    """run_block_eager under a caller's own capture: nothing is uploaded and nothing waited for.  Tensors replaced since the upload are read
    call by call there, and by the next launch outside; the table that a captured launch reads is kept."""
    from paper_2511_15927_amd.decode import BlockDecodeLoop
    cfg = synth.mixer_cfg(2, 8, 12, d_state=4)
    layer = (synth.make_params(cfg, 1, 0), synth.make_params(cfg, 1, 1))
    loop = BlockDecodeLoop(cfg, [layer, layer], 2, device="cpu")
    state, launches, calls, waits = dict(capturing=True), [], [], []
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: state["capturing"])
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: waits.append(state["capturing"]))
    monkeypatch.setattr(bd, "bimamba_block_stack", lambda desc, nl, ns, table, dev, stream=None: launches.append((table, dev)))
    monkeypatch.setattr(bd, "bimamba_block_fwd", lambda *a, stream=None: calls.append(a[3].x.ptr))
    loop.run_block_eager()
    assert len(launches) == 1 and not calls and not waits
    first = launches[0]
    assert first[1].numpy().tobytes() == first[0]
    loop.step_inputs[0]["x"] = torch.zeros_like(loop.step_inputs[0]["x"])
    loop.run_block_eager()
    assert len(launches) == 1 and len(calls) == 4 and calls[0] == loop.step_inputs[0]["x"].data_ptr() and not waits
    state["capturing"] = False
    loop.run_block_eager()
    loop.run_block_eager()
    assert len(launches) == 3 and launches[1][1] is launches[2][1] is not first[1] and waits == [False] and len(calls) == 4
    assert launches[1][0] == launches[1][1].numpy().tobytes() != first[0]
    assert [t is first[1] for t in loop._captured] == [True]


def test_inputs_struct_holds_each_view_as_it_is():
    """Rows, column slices, separate B/C groups, one channel at any stride and empty tensors; a strided channel is refused."""
    base = torch.zeros(3, 7, 40, dtype=torch.bfloat16)
    views = dict(x=base[:, :, 4:20], z=base[:, ::2, 20:36], dt=base[1:, :, 39:], B=base[:, :, :16].unflatten(2, (2, 8)),
                 C=base.transpose(0, 1)[:, :, 8:12].unsqueeze(2))
    got = bd.make_inputs(views)
    for k, t in views.items():
        v = getattr(got, k)
        assert (v.ptr, v.stride_batch, v.stride_token) == (t.data_ptr(), t.stride(0), t.stride(1)), k
    assert bd.make_inputs(dict(views, dt=base[:, :, ::40])).dt.stride_token == 40   # one channel
    assert bd.make_inputs(dict(views, x=base[:0, :, ::2])).x.stride_batch == base.stride(0)
    for bad in (dict(x=base[:, :, ::2]), dict(z=base[0]), dict(B=base[:, :, :32].unflatten(2, (2, 16))[..., :8]), dict(C=base.unflatten(2, (8, 5)).transpose(2, 3))):
        with pytest.raises(AssertionError):
            bd.make_inputs(dict(views, **bad))


def test_stack_form_of_a_table_is_decided_on_the_host():
    """Steps side by side: as many as fit the LDS, in rounds as even as they go; none for a single step, for a descriptor that takes no stack."""
    side = lambda n, *a, **kw: bd.bimamba_block_stack_side_by_side(bd.make_desc(synth.mixer_cfg(*a, **kw)), n)
    assert [side(n, 1, 32, 4096) for n in (-1, 0, 1, 2, 4, 8, 9, 16)] == [0, 0, 0, 0, 4, 8, 5, 8]
    assert side(8, 2, 64, 2045) == 4          # 64 tokens: six steps' LDS, two rounds
    assert side(4, 1, 128, 256) == 0          # long blocks of few channels: time segments
    assert side(8, 1, 32, 64, d_state=32) == side(8, 1, 32, 64, combine=1) == side(8, 0, 32, 64) == 0


def test_copy_inputs_errors_are_decided_on_the_host():
    """bimamba_copy_inputs: missing and narrow views on either side, a place that overlaps a source or another place.  (Legal copies would
    launch: the GPU tests have those.)"""
    Bt, L, Dn, N = 2, 64, 128, 16
    desc = bd.make_desc(synth.mixer_cfg(Bt, L, Dn))
    at = lambda i: 0x1000000 * (i + 1)      # nothing is read
    widths = dict(x=Dn, z=Dn, dt=Dn, B=N, C=N)
    side = lambda i, **over: bd.Inputs(*[over.get(k, bd.Tensor(at(i + j), L * n, n)) for j, (k, n) in enumerate(widths.items())])

    def call(src, dst, desc=desc):
        return bd.lib().bimamba_copy_inputs(C.byref(desc), None if src is None else C.byref(src), None if dst is None else C.byref(dst), None)

    assert call(None, side(5)) == call(side(0), None) == -1
    for k, n in widths.items():
        for bad, code in ((bd.Tensor(None, L * n, n), -1), (bd.Tensor(at(20) + 1, L * n, n), -4), (bd.Tensor(at(20), L * n, n - 1), -2),
                          (bd.Tensor(at(20), L * n - 1, n), -2), (bd.Tensor(at(20), L << 27, 1 << 27), -3)):
            assert call(side(0, **{k: bad}), side(5)) == code, (k, code)
            assert call(side(0), side(5, **{k: bad})) == code, (k, code)
    last = 2 * (Bt * L * Dn - 1)     # the last element of x, in bytes
    for where in (at(0), at(0) + last, at(1), at(3)):      # x's place over x, its end, z, B as they come
        assert call(side(0), side(5, x=bd.Tensor(where, L * Dn, Dn))) == -8, hex(where)
    assert call(side(0), side(5, C=bd.Tensor(at(5) + last, L * N, N))) == -8                   # C's place at the end of x's
    assert call(side(0), side(5, B=bd.Tensor(at(6) - 2 * Bt * L * N + 2, L * N, N))) == -8     # B's place reaches into z's
    assert call(side(0), side(0)) == -8
    assert call(side(0), side(0), bd.make_desc(synth.mixer_cfg(0, L, Dn))) == 0                # nothing to do


def test_step_inputs_of_a_loop_made_in_inference_mode(monkeypatch):
    """Refused outside that mode, as torch refuses every write to such tensors, with nothing written; taken inside it."""
    from paper_2511_15927_amd.decode import BlockDecodeLoop
    cfg = synth.mixer_cfg(1, 4, 8, d_state=4)
    calls = []
    monkeypatch.setattr(bd, "bimamba_copy_inputs", lambda *a, **kw: calls.append(a) or 0)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: -1)
    with torch.inference_mode():
        loop = BlockDecodeLoop(cfg, [(synth.make_params(cfg, 1, 0), synth.make_params(cfg, 1, 1))], 1, device="cpu")
    loop._copies_at_once = True
    given = {k: v.to(torch.bfloat16) for k, v in synth.make_inputs(cfg, 3).items()}
    with pytest.raises(RuntimeError):
        loop.set_step_inputs(0, given)
    assert not calls
    with torch.inference_mode():
        loop.set_step_inputs(0, given)
    assert len(calls) == 1
