"""GPU parity: the HIP path (through the C ABI) against the fp64 oracle, element by element, on seeded inputs.

Tolerances (max over batch elements of relative L2 error): 1e-5 for fp32 I/O, 2e-2 for bf16 I/O with fp32 state.
"""
import numpy as np
import pytest
import torch

from helpers import assert_close, rel_l2, to_np
from paper_2511_15927_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import gpu_util
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return gpu_util


def case(cfg, seed, random_a=False):
    pf, pb = synth.make_params(cfg, seed, 0), synth.make_params(cfg, seed, 1)
    if random_a:
        pf["A"], pb["A"] = synth.random_A(cfg, seed), synth.random_A(cfg, seed + 1)
    return pf, pb, synth.make_inputs(cfg, seed)


def check_fwd(gpu, oracle, cfg, seed, random_a=False, untied=False, sel=None, **override):
    pf, pb, inp = case(cfg, seed, random_a)
    inp_b = synth.make_inputs(cfg, seed + 500) if untied else None
    c = dict(cfg, **override)
    ref = oracle.bimamba_fwd(c, to_np(pf), to_np(pb), to_np(inp), None if inp_b is None else to_np(inp_b), sel=sel)
    runs = [c]
    if c["d_state"] <= 16 and c["seqlen"] <= 256 and c["time_chunks"] == c["state_split"] == 0:
        runs.append(dict(c, time_chunks=1))      # the sweep, where a call left to the library may take the one-launch form
    for r in runs:
        got = gpu.gpu_fwd(r, pf, pb, inp, inp_b)
        assert_close(got if sel is None else got[..., sel], ref, gpu.TOL[c["io"]], r)


def test_cfg0_tiny_fp32(gpu, oracle):
    cfg = synth.CONFIGS["cfg0"]
    check_fwd(gpu, oracle, cfg, synth.config_seed(0))
    check_fwd(gpu, oracle, cfg, synth.config_seed(0), random_a=True)
    check_fwd(gpu, oracle, cfg, synth.config_seed(0), untied=True)
    check_fwd(gpu, oracle, cfg, synth.config_seed(0), combine=synth.COMBINE_SEPARATE)
    check_fwd(gpu, oracle, cfg, synth.config_seed(0), untied=True, combine=synth.COMBINE_SEPARATE, random_a=True)
    check_fwd(gpu, oracle, dict(cfg, dt_softplus=1), synth.config_seed(0))
    check_fwd(gpu, oracle, dict(cfg, io="bf16"), synth.config_seed(0))


def test_cfg0_mamba2_form(gpu, oracle):
    check_fwd(gpu, oracle, synth.CONFIGS["cfg0_m2"], synth.config_seed(0))
    check_fwd(gpu, oracle, dict(synth.CONFIGS["cfg0_m2"], io="bf16"), synth.config_seed(0), untied=True)
    # the paper's 1.3B layer shape: 120 heads x 32, d_state 128, conv over x|B|C
    check_fwd(gpu, oracle, dict(synth.CONFIGS["paper_1p3b"], seqlen=96), 7, sel=list(range(0, 3840, 97)))


@pytest.mark.parametrize("L", [1, 2, 3, 7, 8, 9, 15, 16, 17, 31, 33, 100])
def test_ragged_lengths(gpu, oracle, L):
    for io in ("f32", "bf16"):
        cfg = synth.mixer_cfg(2, L, 96, io=io)
        check_fwd(gpu, oracle, cfg, 100 + L, random_a=True)
        check_fwd(gpu, oracle, cfg, 100 + L, combine=synth.COMBINE_SEPARATE)


@pytest.mark.parametrize("Dn", [1, 24, 63, 64, 65, 200])
def test_ragged_channels(gpu, oracle, Dn):
    cfg = synth.mixer_cfg(3, 37, Dn, io="f32")
    check_fwd(gpu, oracle, cfg, 200 + Dn, random_a=True)


@pytest.mark.parametrize("N", [4, 8, 16, 32, 64, 128])
@pytest.mark.parametrize("a_kind", [0, 1])
def test_state_sizes(gpu, oracle, N, a_kind):
    cfg = synth.mixer_cfg(2, 40, 128, d_state=N, n_heads=128 if a_kind == 0 else 4, a_kind=a_kind, d_kind=a_kind, io="f32")
    check_fwd(gpu, oracle, cfg, 300 + N, random_a=True)


@pytest.mark.parametrize("K", [1, 2, 3, 4])
def test_conv_widths(gpu, oracle, K):
    for L in (1, 2, 5, 19):
        check_fwd(gpu, oracle, synth.mixer_cfg(2, L, 70, d_conv=K, io="f32"), 400 + K)
        check_fwd(gpu, oracle, synth.m2_cfg(1, L, 128, headdim=32, d_state=16, d_conv=K, io="f32"), 410 + K)


def test_groups_and_heads(gpu, oracle):
    cfg = synth.mixer_cfg(2, 50, 256, d_state=16, n_heads=8, n_groups=2, a_kind=1, d_kind=1, conv_bc=1, dt_softplus=1, io="f32")
    check_fwd(gpu, oracle, cfg, 501)
    cfg = synth.mixer_cfg(2, 50, 256, d_state=8, n_heads=256, n_groups=4, io="bf16")
    check_fwd(gpu, oracle, cfg, 502, random_a=True)


@pytest.mark.parametrize("chunks", [1, 2, 3, 5, 8, 64])
def test_time_chunking_matches_oracle(gpu, oracle, chunks):
    cfg = synth.mixer_cfg(2, 203, 130, io="f32", time_chunks=chunks)
    check_fwd(gpu, oracle, cfg, 600, random_a=True)
    check_fwd(gpu, oracle, dict(cfg, combine=1), 600, random_a=True, untied=True)
    m2 = synth.m2_cfg(1, 150, 128, headdim=32, d_state=32, io="f32", time_chunks=chunks)
    check_fwd(gpu, oracle, m2, 601)


@pytest.mark.parametrize("N,split", [(16, 1), (16, 2), (16, 4), (32, 1), (32, 2), (32, 4), (64, 1), (64, 4), (128, 1), (128, 4)])
def test_lanes_per_chain(gpu, oracle, N, split):
    """Every supported way of spreading a chain's states over lanes, on ragged shapes, chunked and not."""
    for io, chunks, L in (("f32", 1, 77), ("bf16", 3, 131), ("f32", 2, 16)):
        cfg = synth.mixer_cfg(2, L, 100, d_state=N, io=io, time_chunks=chunks, state_split=split)
        check_fwd(gpu, oracle, cfg, 900 + N + split, random_a=True)
    m2 = synth.m2_cfg(2, 70, 128, headdim=32, d_state=N, io="f32", state_split=split, time_chunks=2)
    check_fwd(gpu, oracle, m2, 950 + N + split, untied=True)
    sep = synth.mixer_cfg(1, 45, 40, d_state=N, io="f32", combine=1, state_split=split)
    check_fwd(gpu, oracle, sep, 970 + N + split, random_a=True, untied=True)


@pytest.mark.parametrize("kw", [{}, dict(state_split=1, time_chunks=1), dict(state_split=2, time_chunks=1), dict(time_chunks=3)])
def test_strided_views_of_one_projection(gpu, oracle, kw):
    """x, z, dt, B, C as column slices of one [Bt, L, D_in] buffer (channel stride 1, token stride D_in), on the form the
    library picks and on those of the sweep: one launch, lanes split, time segments."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.mixer_cfg(2, 45, 96, io="bf16", **kw)
    pf, pb, inp = case(cfg, 700)
    Dn, N = 96, 16
    widths = dict(z=Dn, x=Dn, B=N, C=N, dt=Dn)
    big = torch.zeros(2, 45, sum(widths.values()) + 5, dtype=torch.bfloat16, device="cuda")
    views, off = {}, 3
    for k in ("z", "x", "B", "C", "dt"):
        views[k] = big[:, :, off:off + widths[k]]
        views[k].copy_(inp[k].reshape(2, 45, -1).to(torch.bfloat16))
        off += widths[k]
    desc = bd.make_desc(cfg)
    out_big = torch.zeros(2, 45, Dn + 7, dtype=torch.bfloat16, device="cuda")
    out = out_big[:, :, 4:4 + Dn]
    dpf, dpb, ws = bd.to_device(pf), bd.to_device(pb), bd.alloc_workspace(desc)
    bd.bimamba_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(views), None, bd.make_tensor(out), ws)
    torch.cuda.synchronize()
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp))
    assert_close(out.float().cpu().numpy(), ref, gpu.TOL["bf16"])
    assert torch.all(out_big[:, :, :4] == 0) and torch.all(out_big[:, :, 4 + Dn:] == 0)


def test_determinism_bitwise(gpu):
    cfg = synth.mixer_cfg(2, 300, 192, io="bf16", time_chunks=3)
    pf, pb, inp = case(cfg, 800)
    a = gpu.gpu_fwd(cfg, pf, pb, inp)
    b = gpu.gpu_fwd(cfg, pf, pb, inp)
    assert np.array_equal(a, b)


def sampled(n, total, seed):
    rng = np.random.default_rng(seed)
    return sorted(rng.choice(total, size=n, replace=False).tolist())


def test_cfg1_1p3b_scale_layer(gpu, oracle):
    cfg = synth.CONFIGS["cfg1"]
    sel = sampled(96, cfg["d_inner"], 1)
    check_fwd(gpu, oracle, cfg, synth.config_seed(1), sel=sel)


def test_cfg1_general_A(gpu, oracle):
    cfg = dict(synth.CONFIGS["cfg1"], batch=2)
    check_fwd(gpu, oracle, cfg, synth.config_seed(1) + 1, random_a=True, sel=sampled(64, 4096, 2))


def test_cfg2_long_sequence(gpu, oracle):
    cfg = synth.CONFIGS["cfg2"]
    check_fwd(gpu, oracle, cfg, synth.config_seed(2), sel=sampled(64, cfg["d_inner"], 3))


def test_headline_shape_sampled(gpu, oracle):
    """d_inner=4096, L=8192, batch 8, bf16: the launch configuration the benchmark times."""
    cfg = synth.CONFIGS["headline"]
    check_fwd(gpu, oracle, cfg, synth.config_seed(9), sel=sampled(24, cfg["d_inner"], 4))


def test_mamba2_shapes_sampled(gpu, oracle):
    cfg = dict(synth.CONFIGS["cfg1_m2"], batch=1, seqlen=1024)
    check_fwd(gpu, oracle, cfg, synth.config_seed(1) + 7, sel=sampled(48, 4096, 5))


def test_cfg4_stack_teacher_forced_per_layer(gpu, oracle):
    """24 mixer layers back to back (layer l's output is layer l+1's x; z, dt, B, C shared; parameters seeded per
    layer).  Every row is independent through the stack, so each layer is checked on sampled channels with the oracle
    fed the GPU's own bf16 input of that layer; the end-to-end drift is reported, not asserted."""
    from paper_2511_15927_amd import binding as bd
    cfg = dict(synth.cfg4(2, 300), io="bf16")
    seed = synth.config_seed(4)
    inp = synth.make_inputs(cfg, seed)
    sel = sampled(24, cfg["d_inner"], 8)
    desc = bd.make_desc(cfg)
    dinp = bd.to_device(inp, cfg)
    ws = bd.alloc_workspace(desc)
    x_gpu = dinp["x"]
    x_ref = inp["x"].numpy().astype(np.float64)[:, :, sel]
    np_in = to_np(inp)
    for layer in range(synth.CFG4_LAYERS):
        pf, pb = synth.make_params(cfg, synth.config_seed(4, layer), 0), synth.make_params(cfg, synth.config_seed(4, layer), 1)
        dpf, dpb = bd.to_device(pf), bd.to_device(pb)
        out = bd.alloc_out(cfg)
        bd.bimamba_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dict(dinp, x=x_gpu)), None,
                       bd.make_tensor(out), ws)
        torch.cuda.synchronize()
        forced = dict(np_in, x=x_gpu.float().cpu().numpy())
        ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), forced, sel=sel)
        got = out.float().cpu().numpy().astype(np.float64)[:, :, sel]
        assert_close(got, ref, gpu.TOL["bf16"], layer)
        x_gpu = out


@pytest.mark.parametrize("N,split", [(16, 1), (16, 2), (16, 4), (32, 2), (8, 1)])
def test_decay_progression_detected_path(gpu, oracle, N, split):
    """A[h, n] arithmetic in n with a different start and step per channel (the form the library detects on the device
    and evaluates with two exponentials per token), and the same A with one entry nudged so that detection must fail:
    both must match the oracle (bf16 I/O, long enough for detection to be attempted, chunked and not)."""
    for chunks in (1, 3):
        cfg = synth.mixer_cfg(2, 300, 136, d_state=N, io="bf16", state_split=split, time_chunks=chunks)
        pf, pb, inp = case(cfg, 1500 + N)
        hidx = torch.arange(cfg["n_heads"], dtype=torch.float32)
        n = torch.arange(N, dtype=torch.float32)
        for p, sign in ((pf, 1.0), (pb, 2.0)):
            start = -(0.5 + 0.25 * (hidx % 7))                 # multiples of 1/4: every entry is exact in fp32
            step = -(0.125 * sign) * (1 + hidx % 3)
            p["A"] = (start[:, None] + n[None, :] * step[:, None]).contiguous()
        ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp))
        assert_close(gpu.gpu_fwd(cfg, pf, pb, inp), ref, gpu.TOL["bf16"])
        pf2 = dict(pf, A=pf["A"].clone())
        pf2["A"][5, N - 1] *= 1.0 + 2.0 ** -20                  # no longer a progression: the general path must run
        ref2 = oracle.bimamba_fwd(cfg, to_np(pf2), to_np(pb), to_np(inp))
        assert_close(gpu.gpu_fwd(cfg, pf2, pb, inp), ref2, gpu.TOL["bf16"])


def test_large_batch_shallow_tile(gpu, oracle):
    """Enough chains for four waves per SIMD: the library switches to the shallow-tile instantiation."""
    for L, ra in ((100, True), (37, False)):
        cfg = synth.mixer_cfg(32, L, 4096)
        check_fwd(gpu, oracle, cfg, 1600 + L, random_a=ra, sel=sampled(16, 4096, 9))


@pytest.mark.parametrize("Dn,split", [(192, 1), (96, 2), (48, 4), (320, 1), (160, 2)])
def test_odd_number_of_channel_tiles(gpu, oracle, Dn, split):
    """A workgroup covers two channel tiles; with an odd number of tiles the last workgroup's second pair of waves
    shadows the first (same values to the same addresses).  Whole sequence and time segments, with a committed state."""
    N = 64 if split == 4 else 16
    for chunks in (1, 3):
        cfg = synth.mixer_cfg(3, 75, Dn, d_state=N, io="f32", state_split=split, time_chunks=chunks)
        check_fwd(gpu, oracle, cfg, 1700 + Dn + chunks)
    cfg = synth.mixer_cfg(2, 40, Dn, d_state=N, io="f32", state_split=split)
    pf, pb, inp = case(cfg, 1750 + Dn)
    ref, h_ref, _ = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), want_tail=False)
    got, h_got, _ = gpu.gpu_block_fwd(cfg, pf, pb, inp)
    assert_close(got, ref, gpu.TOL["f32"])
    assert rel_l2(h_got, h_ref) < 1e-5


@pytest.mark.parametrize("batch,L", [(8, 300), (11, 150), (13, 130), (9, 520), (40, 70)])
def test_launch_geometries_of_the_batch_sweep(gpu, oracle, batch, L):
    """Shapes on either side of each geometry rule at d_inner 4096: two lanes per chain in one round, time segments,
    one lane per chain from 1.5 waves per SIMD, more than one round of workgroups (no turns), sampled channels."""
    cfg = synth.mixer_cfg(batch, L, 4096)
    check_fwd(gpu, oracle, cfg, 1800 + batch, sel=sampled(16, 4096, batch))


@pytest.mark.parametrize("kw", [{}, dict(state_split=1, time_chunks=1), dict(state_split=2, time_chunks=1)])
def test_output_as_a_column_slice_of_the_inputs_buffer(gpu, oracle, kw):
    """out may live in the same buffer as the inputs as long as its columns stay apart from theirs (same strides): the
    host's overlap check accepts it and no input column is disturbed; an out that runs into z is refused."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.mixer_cfg(2, 45, 96, io="bf16", **kw)
    pf, pb, inp = case(cfg, 710)
    Dn, N = 96, 16
    widths = dict(z=Dn, x=Dn, B=N, C=N, dt=Dn, out=Dn)
    pitch = sum(widths.values()) + 8
    big = torch.zeros(2, 45, pitch, dtype=torch.bfloat16, device="cuda")
    views, off = {}, 0
    for k in ("z", "x", "B", "C", "dt", "out"):
        views[k] = big[:, :, off:off + widths[k]]
        if k != "out":
            views[k].copy_(inp[k].reshape(2, 45, -1).to(torch.bfloat16))
        off += widths[k]
    before = big.clone()
    desc = bd.make_desc(cfg)
    dpf, dpb, ws = bd.to_device(pf), bd.to_device(pb), bd.alloc_workspace(desc)
    args = (desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(views), None)
    bd.bimamba_fwd(*args, bd.make_tensor(views["out"]), ws)
    torch.cuda.synchronize()
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp))
    assert_close(views["out"].float().cpu().numpy(), ref, gpu.TOL["bf16"])
    keep = [c for c in range(pitch) if not (off - Dn <= c < off)]
    assert torch.equal(big[:, :, keep], before[:, :, keep])
    clash = big[:, :, Dn // 2:Dn // 2 + Dn]                       # straddles z and x
    assert bd.bimamba_fwd(*args, bd.make_tensor(clash), ws, check=False) == -8


@pytest.mark.parametrize("batch,L,Dn,N,io", [
    (5, 170, 1600, 16, "f32"),       # too short to cut: two lanes per chain, whole
    (1, 257, 512, 16, "f32"), (1, 1101, 72, 16, "bf16"), (2, 9001, 40, 16, "bf16"),    # too narrow for a round of segments
    (1, 1928, 200, 8, "bf16"), (2, 700, 40, 4, "f32"), (1, 5003, 64, 8, "f32"),
    (2, 777, 320, 16, "bf16"),       # two lanes per chain, segments of 24 tokens or more, a ragged last one
    (1, 2051, 640, 16, "f32"),       # the same with a few tokens more than whole segments
    (1, 3001, 1024, 16, "bf16"),     # one round of one-lane segments
    (4, 8191, 192, 16, "bf16"),      # four rounds
    (3, 900, 3072, 16, "f32"),       # whole: two waves per SIMD at most
    (1, 300, 512, 8, "f32"), (2, 530, 640, 8, "bf16"), (1, 1601, 456, 4, "f32")])   # no lane splitting below 16 states
@pytest.mark.parametrize("combine", [0, 1])
def test_geometry_left_to_the_library(gpu, oracle, batch, L, Dn, N, io, combine):
    """Every kind of geometry the cost rule picks, against the oracle, and against one segment with one lane per chain."""
    cfg = synth.mixer_cfg(batch, L, Dn, d_state=N, io=io, combine=combine)
    pf, pb = synth.make_params(cfg, L, 0), synth.make_params(cfg, L, 1)
    if L % 2:
        pf["A"], pb["A"] = synth.random_A(cfg, L), synth.random_A(cfg, L + 1)
    inp = synth.make_inputs(cfg, L)
    sel = sorted(np.random.default_rng(L).choice(Dn, size=24, replace=False).tolist())
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), sel=sel)
    assert_close(gpu.gpu_fwd(cfg, pf, pb, inp)[..., sel], ref, gpu.TOL[io])
    assert_close(gpu.gpu_fwd(cfg, pf, pb, inp, state_split=1, time_chunks=1)[..., sel], ref, gpu.TOL[io])
