"""GPU parity of the chunked matrix-core path for the Mamba-2 parameterisation (bf16 I/O, one decay rate per head)
against the fp64 oracle, and against the lane-per-chain kernels it replaces for these shapes."""
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


def case(cfg, seed):
    return synth.make_params(cfg, seed, 0), synth.make_params(cfg, seed, 1), synth.make_inputs(cfg, seed)


@pytest.mark.parametrize("N,P", [(128, 64), (128, 32), (64, 64), (64, 32)])
@pytest.mark.parametrize("L", [1, 40, 64, 65, 200])
def test_ssd_matches_oracle(gpu, oracle, N, P, L):
    cfg = synth.m2_cfg(2, L, 4 * P, headdim=P, d_state=N)
    pf, pb, inp = case(cfg, 1000 + N + P + L)
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp))
    got = gpu.gpu_fwd(cfg, pf, pb, inp)
    assert_close(got, ref, gpu.TOL["bf16"])
    # the lane-per-chain kernels on the same inputs (forced by state_split) agree with the same oracle
    got_valu = gpu.gpu_fwd(cfg, pf, pb, inp, state_split=1)
    assert_close(got_valu, ref, gpu.TOL["bf16"])


@pytest.mark.parametrize("kw", [
    dict(combine=1), dict(conv_bc=0), dict(dt_softplus=0), dict(d_kind=0), dict(d_conv=2), dict(n_groups=2),
    dict(combine=1, conv_bc=0, dt_softplus=0, d_kind=0, d_conv=3),
])
def test_ssd_option_coverage(gpu, oracle, kw):
    cfg = synth.m2_cfg(2, 150, 256, headdim=64, d_state=64, **kw)
    pf, pb, inp = case(cfg, 1100)
    inp_b = synth.make_inputs(cfg, 1101)
    for other in (None, inp_b):
        ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), None if other is None else to_np(other))
        got = gpu.gpu_fwd(cfg, pf, pb, inp, other)
        assert_close(got, ref, gpu.TOL["bf16"], (kw, other is not None))


def test_ssd_long_sequence_state_stays_fp32(gpu, oracle):
    """Many chunks: the state is carried in fp32 accumulators for the whole sequence."""
    cfg = synth.m2_cfg(1, 4096, 256, headdim=64, d_state=128)
    pf, pb, inp = case(cfg, 1200)
    sel = list(range(0, 256, 5))
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), sel=sel)
    got = gpu.gpu_fwd(cfg, pf, pb, inp)[..., sel]
    assert_close(got, ref, gpu.TOL["bf16"])


def test_ssd_block_variant_carries_state_and_tail(gpu, oracle):
    cfg = synth.m2_cfg(2, 96, 128, headdim=32, d_state=64)
    pf, pb, inp = case(cfg, 1300)
    K, Dn, GN = cfg["d_conv"], cfg["d_inner"], cfg["n_groups"] * cfg["d_state"]
    g_full, h_full = oracle.one_direction(cfg, to_np(pf), to_np(inp), +1)
    h, tail = None, None
    h_ref, tail_ref = None, None
    for t0, t1 in ((0, 32), (32, 35), (35, 96)):
        blk = {k: v[:, t0:t1].contiguous() for k, v in inp.items()}
        cb = dict(cfg, seqlen=t1 - t0)
        ref, h_ref, tail_ref = oracle.bimamba_block_fwd(cb, to_np(pf), to_np(pb), to_np(blk), h_in=h_ref, tail_in=tail_ref)
        out, h, tail = gpu.gpu_block_fwd(cb, pf, pb, blk, h_in=h, tail_in=tail)
        assert_close(out, ref, gpu.TOL["bf16"], (t0, t1))
        assert np.array_equal(tail, tail_ref)
        # the chain of GPU states follows the oracle's chain (bf16 operand rounding accumulates only mildly)
        assert rel_l2(h, h_ref) < 1e-2, (t0, t1)
    assert rel_l2(h, h_full) < 1e-2


def test_ssd_benchmark_shapes_sampled(gpu, oracle):
    for name, L in (("cfg1_m2", 2048), ("paper_1p3b", 1024)):
        cfg = dict(synth.CONFIGS[name], batch=2, seqlen=L)
        pf, pb, inp = case(cfg, 1400)
        sel = sorted(np.random.default_rng(3).choice(cfg["d_inner"], size=48, replace=False).tolist())
        ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), sel=sel)
        got = gpu.gpu_fwd(cfg, pf, pb, inp)[..., sel]
        assert_close(got, ref, gpu.TOL["bf16"], name)


@pytest.mark.parametrize("lead", [4, 3])
def test_ssd_strided_views_and_unaligned_fallback(gpu, oracle, lead):
    """Inputs as column slices of one projection buffer.  The chunked kernels read x as channel pairs: with an even
    column offset and even row pitch they run; with an odd offset the call must still succeed (lane-per-chain
    kernels take over inside the same workspace) and give the same answer."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.m2_cfg(2, 150, 128, headdim=64, d_state=64)
    pf, pb, inp = case(cfg, 1500)
    Bt, L, Dn, H, GN = 2, 150, 128, 2, 64
    widths = dict(z=Dn, x=Dn, B=GN, C=GN, dt=H)
    pitch = lead + sum(widths.values()) + 6
    big = torch.zeros(Bt, L, pitch, dtype=torch.bfloat16, device="cuda")
    views, off = {}, lead
    for k in ("z", "x", "B", "C", "dt"):
        views[k] = big[:, :, off:off + widths[k]]
        views[k].copy_(inp[k].reshape(Bt, L, -1).to(torch.bfloat16))
        off += widths[k]
    assert (views["x"].data_ptr() % 4 == 0) == (lead % 2 == 0)
    desc = bd.make_desc(cfg)
    out_big = torch.zeros(Bt, L, Dn + 8, dtype=torch.bfloat16, device="cuda")
    out = out_big[:, :, 4:4 + Dn]
    dpf, dpb, ws = bd.to_device(pf), bd.to_device(pb), bd.alloc_workspace(desc)
    bd.bimamba_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(views), None, bd.make_tensor(out), ws)
    torch.cuda.synchronize()
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp))
    assert_close(out.float().cpu().numpy(), ref, gpu.TOL["bf16"])
    assert torch.all(out_big[:, :, :4] == 0) and torch.all(out_big[:, :, 4 + Dn:] == 0)


@pytest.mark.parametrize("L", [40, 130])
def test_ssd_more_items_than_compute_units(gpu, oracle, L):
    """More (batch, head) pairs than the chip has CUs (several rounds of workgroups), one and three chunks each: the
    full-sequence call, and a block call that loads and commits every pair's state."""
    cfg = synth.m2_cfg(3, L, 32 * 200, headdim=32, d_state=64)       # 600 items, one or three chunks each
    pf, pb, inp = case(cfg, 1600 + L)
    sel = sorted(np.random.default_rng(5).choice(cfg["d_inner"], size=300, replace=False).tolist())
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), sel=sel)
    got = gpu.gpu_fwd(cfg, pf, pb, inp)[..., sel]
    assert_close(got, ref, gpu.TOL["bf16"])
    g = torch.Generator().manual_seed(L)
    h0 = (0.2 * torch.randn(3, cfg["d_inner"], 64, generator=g)).float()
    tail0 = synth.round_io(torch.randn(3, 3, cfg["d_inner"] + 128, generator=g), "bf16")
    ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), h_in=h0.numpy(), tail_in=tail0.numpy())
    out, h, tail = gpu.gpu_block_fwd(cfg, pf, pb, inp, h_in=h0, tail_in=tail0)
    assert_close(out, ref, gpu.TOL["bf16"])
    assert rel_l2(h, h_ref) < 1e-2
    assert np.array_equal(tail, t_ref)


def test_ssd_state_not_16_byte_aligned_falls_back(gpu, oracle):
    """The matrix-core kernels move the cached state as 16-byte pieces.  A state buffer that is only 4-byte aligned
    must still work: the call runs on the lane-per-chain kernels inside the same workspace."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.m2_cfg(2, 70, 128, headdim=64, d_state=64)
    pf, pb, inp = case(cfg, 1700)
    g = torch.Generator().manual_seed(3)
    h0 = (0.2 * torch.randn(2, 128, 64, generator=g)).float()
    ref, h_ref, _ = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), h_in=h0.numpy(), want_tail=False)
    n = h0.numel()
    buf_in = torch.zeros(n + 1, dtype=torch.float32, device="cuda")
    buf_out = torch.zeros(n + 1, dtype=torch.float32, device="cuda")
    h_in, h_out = buf_in[1:].view(2, 128, 64), buf_out[1:].view(2, 128, 64)
    h_in.copy_(h0)
    assert h_in.data_ptr() % 16 == 4
    desc = bd.make_desc(cfg)
    dpf, dpb, dinp = bd.to_device(pf), bd.to_device(pb), bd.to_device(inp, cfg)
    out, ws = bd.alloc_out(cfg), bd.alloc_workspace(desc, 1)
    bd.bimamba_block_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp), None, h_in, None, h_out,
                         None, bd.make_tensor(out), ws)
    torch.cuda.synchronize()
    assert_close(out.float().cpu().numpy(), ref, gpu.TOL["bf16"])
    assert rel_l2(h_out.cpu().numpy(), h_ref) < 1e-5      # the lane-per-chain kernels keep the state to fp32 accuracy
    assert float(buf_out[0]) == 0.0


@pytest.mark.parametrize("L,batch,N,parts,kw", [(1550, 1, 128, 3, {}), (2117, 2, 64, 4, dict(combine=1)), (1100, 1, 128, 2, dict(combine=1)),
                                                (1481, 1, 64, 3, dict(conv_bc=0, dt_softplus=0, d_kind=0))])
def test_ssd_time_parts(gpu, oracle, L, batch, N, parts, kw):
    """Few (batch, head) items and many chunks: each item's chunks are dealt to several workgroups (a state-only pass,
    a carry over the parts, then the output pass).  Ragged last part, both combines, and the block variant: the parts
    start from the cached state and the committed state is the last part's."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.m2_cfg(batch, L, 256, headdim=64, d_state=N, **kw)
    assert bd.bimamba_time_chunks(bd.make_desc(cfg)) == parts
    pf, pb, inp = case(cfg, 1900 + L)
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp))
    assert_close(gpu.gpu_fwd(cfg, pf, pb, inp), ref, gpu.TOL["bf16"])
    # block variant on top of a prefix
    m = 5
    pre = {k: v[:, :m].contiguous() for k, v in inp.items()}
    blk = {k: v[:, m:].contiguous() for k, v in inp.items()}
    _, h_pre, tail_pre = oracle.bimamba_block_fwd(dict(cfg, seqlen=m), to_np(pf), to_np(pb), to_np(pre))
    cb = dict(cfg, seqlen=L - m)
    assert bd.bimamba_time_chunks(bd.make_desc(cb)) == parts
    ref_b, h_ref, tail_ref = oracle.bimamba_block_fwd(cb, to_np(pf), to_np(pb), to_np(blk), h_in=h_pre.astype(np.float32), tail_in=tail_pre)
    out, h, tail = gpu.gpu_block_fwd(cb, pf, pb, blk, h_in=h_pre.astype(np.float32), tail_in=tail_pre)
    assert_close(out, ref_b, gpu.TOL["bf16"])
    assert rel_l2(h, h_ref) < 1e-2
    assert np.array_equal(tail, tail_ref)


@pytest.mark.parametrize("token_stride", [1 << 24, (1 << 24) + 2])
@pytest.mark.parametrize("combine", [0, 1])
def test_ssd_time_parts_with_a_wide_x_stride(gpu, oracle, token_stride, combine):
    """x as a view with a token stride of 2^24 elements, the widest for which the state pass of the time parts may
    address a chunk's rows with 32-bit offsets, and just beyond it, where the call runs without parts.  (Directions kept apart: those that
    are added meet in the middle, whatever the stride.)"""
    from paper_2511_15927_amd import binding as bd
    L = 1030
    cfg = synth.m2_cfg(1, L, 256, headdim=64, d_state=64, combine=combine)
    assert bd.bimamba_time_chunks(bd.make_desc(cfg)) == 1 + combine
    pf, pb, inp = case(cfg, 4242)
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp))
    desc = bd.make_desc(cfg)
    dpf, dpb, dinp = bd.to_device(pf), bd.to_device(pb), bd.to_device(inp, cfg)
    big = torch.empty((L - 1) * token_stride + 256, dtype=torch.bfloat16, device="cuda")
    wide = big.as_strided((1, L, 256), (0, token_stride, 1))
    wide.copy_(dinp["x"])
    dinp["x"] = wide
    out, ws = bd.alloc_out(cfg), bd.alloc_workspace(desc)
    bd.bimamba_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp), None, bd.make_tensor(out), ws)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().reshape(ref.shape)
    del big, wide, dinp
    torch.cuda.empty_cache()
    assert_close(got, ref, gpu.TOL["bf16"])


@pytest.mark.parametrize("N,headdim,combine,own", [(128, 64, 0, False), (128, 32, 0, True), (64, 32, 1, False), (64, 64, 0, True)])
def test_ssd_time_parts_down_to_one_short_chunk(gpu, oracle, N, headdim, combine, own):
    """41 chunks in parts of ten, the last part one chunk of five tokens: every head width, z shared (gated once, behind the sum) and
    the reverse direction's own, the halves added and kept apart."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.m2_cfg(1, 2565, 256, headdim=headdim, d_state=N, combine=combine)
    assert bd.bimamba_time_chunks(bd.make_desc(cfg)) == 5
    pf, pb, inp = case(cfg, 2565 + N)
    other = synth.make_inputs(cfg, 2566) if own else None
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), None if other is None else to_np(other))
    assert_close(gpu.gpu_fwd(cfg, pf, pb, inp, other), ref, gpu.TOL["bf16"])


def test_ssd_rows_too_far_apart_for_time_parts(gpu, oracle):
    """z as a view with a token stride beyond 2^24 elements, the widest whose rows in a chunk 32-bit offsets reach: in time parts like
    any other call, every row addressed by itself."""
    from paper_2511_15927_amd import binding as bd
    L, token_stride = 1030, (1 << 24) + 2
    cfg = synth.m2_cfg(1, L, 256, headdim=64, d_state=64)
    pf, pb, inp = case(cfg, 4243)
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp))
    desc = bd.make_desc(cfg)
    dpf, dpb, dinp = bd.to_device(pf), bd.to_device(pb), bd.to_device(inp, cfg)
    big = torch.empty((L - 1) * token_stride + 256, dtype=torch.bfloat16, device="cuda")
    wide = big.as_strided((1, L, 256), (0, token_stride, 1))
    wide.copy_(dinp["z"])
    dinp["z"] = wide
    out, ws = bd.alloc_out(cfg), bd.alloc_workspace(desc)
    bd.bimamba_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp), None, bd.make_tensor(out), ws)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    del big, wide, dinp
    torch.cuda.empty_cache()
    assert_close(got, ref, gpu.TOL["bf16"])


@pytest.mark.parametrize("L,combine,views", [(1030, 0, ("out",)), (2050, 0, ("z", "x")), (150, 0, ("z",)), (131, 1, ("out", "z")), (150, 0, ("z", "x", "out"))])
def test_ssd_block_call_with_rows_far_apart(gpu, oracle, L, combine, views):
    """z, out or x as views with token strides beyond 2^24 elements, with and without time parts (x that far apart: none), as a block call
    from a cached state and tail, which it commits; activations per direction, so that one of them is near."""
    from paper_2511_15927_amd import binding as bd
    stride = (1 << 24) + 2
    cfg = synth.m2_cfg(1, L, 128, headdim=64, d_state=64, combine=combine)
    pf, pb, inp = case(cfg, 4300 + L)
    inp_b = synth.make_inputs(cfg, 4400 + L)
    K, Dn, N = cfg["d_conv"], cfg["d_inner"], cfg["d_state"]
    g = torch.Generator().manual_seed(L)
    h0 = (0.2 * torch.randn(1, Dn, N, generator=g)).float()
    tail0 = synth.round_io(torch.randn(1, K - 1, synth.conv_channels(cfg), generator=g), "bf16")
    ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), to_np(inp_b), h_in=h0.numpy(), tail_in=tail0.numpy())
    desc = bd.make_desc(cfg)
    dpf, dpb, dinp, dinp_b = bd.to_device(pf), bd.to_device(pb), bd.to_device(inp, cfg), bd.to_device(inp_b, cfg)
    # one buffer, the views beside each other in its rows
    big = torch.empty((L - 1) * stride + 1024, dtype=torch.bfloat16, device="cuda")
    out, place = bd.alloc_out(cfg), 0
    for v in views:
        t = out if v == "out" else dinp[v]
        wide = big.as_strided(t.shape, (0, stride, 1), place)
        place += t.shape[2]
        if v == "out":
            out = wide
        else:
            wide.copy_(t)
            dinp[v] = wide
    h, tail = h0.cuda(), tail0.to(torch.bfloat16).cuda()
    ws = bd.alloc_workspace(desc, 1)
    bd.bimamba_block_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp), bd.make_inputs(dinp_b), h, tail, h, tail,
                         bd.make_tensor(out), ws)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    del big, out, dinp
    torch.cuda.empty_cache()
    assert_close(got.reshape(ref.shape), ref, gpu.TOL["bf16"])
    assert rel_l2(h.cpu().numpy(), h_ref) < 1e-2
    assert np.array_equal(tail.float().cpu().numpy(), t_ref)


@pytest.mark.parametrize("name,batch,combine,parts", [("cfg2_m2", 1, 0, 4), ("headline_m2", 1, 0, 4), ("headline_m2", 1, 1, 2), ("headline_m2", 2, 0, 1)])
def test_ssd_time_parts_at_benchmark_size_sampled(gpu, oracle, name, batch, combine, parts):
    """The time-part path (state pass over sub-parts, carry, concurrent output pass) at the benchmark's own sizes, in the
    launch configuration the benchmark times; with two parts at most the added directions meet in the middle instead.  The oracle
    runs on sampled channels."""
    from paper_2511_15927_amd import binding as bd
    cfg = dict(synth.CONFIGS[name], batch=batch, combine=combine)
    assert bd.bimamba_time_chunks(bd.make_desc(cfg)) == parts
    pf, pb, inp = case(cfg, 1700 + batch)
    sel = sorted(np.random.default_rng(5).choice(cfg["d_inner"], size=24, replace=False).tolist())
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), sel=sel)
    got = gpu.gpu_fwd(cfg, pf, pb, inp)[..., sel]
    assert_close(got, ref, gpu.TOL["bf16"], name)


def test_ssd_block_call_at_benchmark_size_sampled(gpu, oracle):
    """A block-diffusion step at the benchmark's size (batch 16, 32 tokens, 64 heads x 64, N 128) from a cached state and
    conv tail: one scan launch runs both directions of every (batch, head) item; sampled channels against the oracle,
    the committed state of those channels and the whole committed tail."""
    cfg = synth.CONFIGS["cfg3_block_m2"]
    pf, pb, inp = case(cfg, 1800)
    Bt, Dn, N, K = cfg["batch"], cfg["d_inner"], cfg["d_state"], cfg["d_conv"]
    tail_ch = synth.conv_channels(cfg)
    g = torch.Generator().manual_seed(1801)
    h0 = (0.2 * torch.randn(Bt, Dn, N, generator=g)).float()
    tail0 = synth.round_io(torch.randn(Bt, K - 1, tail_ch, generator=g), cfg["io"])
    sel = sorted(np.random.default_rng(6).choice(Dn, size=48, replace=False).tolist())
    ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), h_in=h0.numpy(), tail_in=tail0.numpy(), sel=sel)
    out, h, tail = gpu.gpu_block_fwd(cfg, pf, pb, inp, h_in=h0, tail_in=tail0)
    assert_close(out[..., sel], ref, gpu.TOL["bf16"])
    assert rel_l2(h[:, sel, :], h_ref[:, sel, :]) < 1e-2
    assert np.array_equal(tail, t_ref)


@pytest.mark.parametrize("L,batch,heads,headdim,N", [(65, 1, 3, 64, 128), (130, 3, 8, 32, 64), (1100, 2, 4, 64, 64), (1157, 1, 5, 32, 128)])
@pytest.mark.parametrize("wide_z", [False, True])
def test_ssd_both_directions_in_one_launch(gpu, oracle, L, batch, heads, headdim, N, wide_z):
    """Output halves kept apart, activations per direction: both directions walk in one launch, with and without time
    parts; a z token stride beyond 2^24 elements takes the form that addresses every row by itself."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.m2_cfg(batch, L, heads * headdim, headdim=headdim, d_state=N, combine=synth.COMBINE_SEPARATE)
    pf, pb, inp = case(cfg, 2100 + L)
    inp_b = synth.make_inputs(cfg, 2600 + L)
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), to_np(inp_b))
    if not wide_z:
        assert_close(gpu.gpu_fwd(cfg, pf, pb, inp, inp_b), ref, gpu.TOL["bf16"])
        return
    if L > 200 or batch > 1:
        pytest.skip("one small call is enough for the strided view")
    stride = (1 << 24) + 2
    desc = bd.make_desc(cfg)
    dpf, dpb, dinp, dinp_b = bd.to_device(pf), bd.to_device(pb), bd.to_device(inp, cfg), bd.to_device(inp_b, cfg)
    z = torch.empty((L - 1) * stride + cfg["d_inner"], dtype=torch.bfloat16, device="cuda").as_strided((1, L, cfg["d_inner"]), (0, stride, 1))
    z.copy_(dinp["z"])
    dinp["z"] = z
    out, ws = bd.alloc_out(cfg), bd.alloc_workspace(desc)
    bd.bimamba_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp), bd.make_inputs(dinp_b), bd.make_tensor(out), ws)
    torch.cuda.synchronize()
    assert_close(out.float().cpu().numpy().reshape(ref.shape), ref, gpu.TOL["bf16"])


@pytest.mark.parametrize("N,P", [(128, 64), (128, 32), (64, 64), (64, 32)])
@pytest.mark.parametrize("L,heads,groups,kw", [
    (65, 130, 1, {}),                              # two chunks, the second of one token; two heads to a workgroup
    (200, 132, 2, dict(d_conv=3)),                 # four chunks, two groups
    (130, 131, 1, dict(d_kind=0)),                 # three chunks, an odd head count: one head to a workgroup
])
def test_ssd_wide_forms(gpu, oracle, N, P, L, heads, groups, kw):
    """Enough (batch, head) items for the many-wave walk in both of its forms, as a block call from a cached state and tail
    (the state and the tail are committed), with the parked result gated and ungated, and with output halves kept apart."""
    cfg = synth.m2_cfg(2, L, heads * P, headdim=P, d_state=N, n_groups=groups, **kw)
    pf, pb, inp = case(cfg, 3100 + L + N + P)
    g = torch.Generator().manual_seed(L + P)
    K, Dn = cfg["d_conv"], cfg["d_inner"]
    h0 = (0.2 * torch.randn(2, Dn, N, generator=g)).float()
    tail0 = synth.round_io(torch.randn(2, K - 1, synth.conv_channels(cfg), generator=g), "bf16")
    sel = sorted(np.random.default_rng(L).choice(Dn, size=40, replace=False).tolist() + [0, Dn - 1])
    inp_b = dict(inp, z=synth.make_inputs(cfg, 3200 + L)["z"])
    for combine, other in ((0, None), (0, inp_b), (1, inp_b)):
        c = dict(cfg, combine=combine)
        ref, h_ref, t_ref = oracle.bimamba_block_fwd(c, to_np(pf), to_np(pb), to_np(inp), None if other is None else to_np(other),
                                                     h_in=h0.numpy(), tail_in=tail0.numpy(), sel=sel)
        out, h, tail = gpu.gpu_block_fwd(c, pf, pb, inp, other, h_in=h0, tail_in=tail0)
        assert_close(out[..., sel], ref, gpu.TOL["bf16"], (combine, other is not None))
        assert rel_l2(h[:, sel, :], h_ref[:, sel, :]) < 1e-2
        assert np.array_equal(tail, t_ref)


@pytest.mark.parametrize("heads", [4, 260])
def test_ssd_wide_fast_decay_and_odd_pitch(gpu, oracle, heads):
    """Chunks that decay by more than 2^100 (per-element decay factors), and z and out that are not aligned channel pairs."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.m2_cfg(1, 150, heads * 32, headdim=32, d_state=64)
    pf, pb, inp = case(cfg, 3300)
    for p in (pf, pb):
        p["A"] = p["A"] * torch.where(torch.arange(heads) % 2 == 0, 40.0, 1.0)
    ref = oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp))
    assert_close(gpu.gpu_fwd(cfg, pf, pb, inp), ref, gpu.TOL["bf16"])
    Dn = cfg["d_inner"]
    dinp = bd.to_device(inp, cfg)
    z = torch.empty(1, 150, Dn + 3, dtype=torch.bfloat16, device="cuda")[:, :, 1:1 + Dn]
    z.copy_(dinp["z"])
    dinp["z"] = z
    big = torch.zeros(1, 150, Dn + 5, dtype=torch.bfloat16, device="cuda")
    out = big[:, :, 2:2 + Dn]
    desc, dpf, dpb = bd.make_desc(cfg), bd.to_device(pf), bd.to_device(pb)
    bd.bimamba_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp), None, bd.make_tensor(out), bd.alloc_workspace(desc))
    torch.cuda.synchronize()
    assert_close(out.float().cpu().numpy(), ref, gpu.TOL["bf16"])
    assert torch.all(big[:, :, :2] == 0) and torch.all(big[:, :, 2 + Dn:] == 0)


@pytest.mark.parametrize("L", [1, 3, 31, 32, 33, 63, 64])
@pytest.mark.parametrize("N,P,heads,groups,kw", [
    (128, 64, 3, 1, {}),
    (128, 32, 3, 1, dict(d_conv=2)),                  # a last workgroup of half its channels
    (64, 32, 5, 1, dict(d_kind=0, d_conv=1)),
    (64, 64, 4, 2, dict(conv_bc=0, dt_softplus=0)),
])
def test_ssd_one_chunk_calls(gpu, oracle, L, N, P, heads, groups, kw):
    """Block steps around the 32-token blocks: from a cached state and tail and from none, committed in place, shared and separate
    activations, both combines; a decay too fast for separable factors; views at odd places."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.m2_cfg(2, L, heads * P, headdim=P, d_state=N, n_groups=groups, **kw)
    pf, pb, inp = case(cfg, 3400 + L + N + P)
    for p in (pf, pb):
        p["A"] = p["A"] * torch.where(torch.arange(heads) % 3 == 1, 60.0, 1.0)
    other = synth.make_inputs(cfg, 3500 + L)
    K, Dn, ch = cfg["d_conv"], cfg["d_inner"], synth.conv_channels(cfg)
    g = torch.Generator().manual_seed(L + P)
    h0 = (0.2 * torch.randn(2, Dn, N, generator=g)).float()
    tail0 = synth.round_io(torch.randn(2, K - 1, ch, generator=g), "bf16") if K > 1 else None
    for combine, in_b, start in ((0, None, True), (0, other, True), (1, other, False), (1, dict(inp, z=other["z"]), True)):
        c = dict(cfg, combine=combine)
        ref, h_ref, t_ref = oracle.bimamba_block_fwd(c, to_np(pf), to_np(pb), to_np(inp), None if in_b is None else to_np(in_b),
                                                     h_in=h0.numpy() if start else None, tail_in=tail0.numpy() if start and K > 1 else None)
        out, h, tail = gpu.gpu_block_fwd(c, pf, pb, inp, in_b, h_in=h0 if start else None, tail_in=tail0 if start else None)
        assert_close(out, ref, gpu.TOL["bf16"], (combine, in_b is not None))
        assert rel_l2(h, h_ref) < 1e-2
        if K > 1:
            assert np.array_equal(tail, t_ref)
    # in place, from columns of wider buffers
    ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), h_in=h0.numpy(), tail_in=tail0.numpy() if K > 1 else None)
    dinp, desc, dpf, dpb = bd.to_device(inp, cfg), bd.make_desc(cfg), bd.to_device(pf), bd.to_device(pb)
    for k, off in (("x", 2), ("z", 3)):
        wide = torch.full((2, L, Dn + 6), 7.0, dtype=torch.bfloat16, device="cuda")[:, :, off:off + Dn]
        wide.copy_(dinp[k])
        dinp[k] = wide
    big = torch.zeros(2, L, Dn + 3, dtype=torch.bfloat16, device="cuda")
    h, tail = h0.cuda(), tail0.to(torch.bfloat16).cuda() if K > 1 else None
    bd.bimamba_block_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp), None, h, tail, h, tail,
                         bd.make_tensor(big[:, :, 1:1 + Dn]), bd.alloc_workspace(desc, 1))
    torch.cuda.synchronize()
    if K > 1:
        assert np.array_equal(tail.float().cpu().numpy(), t_ref)
    assert_close(big[:, :, 1:1 + Dn].float().cpu().numpy(), ref, gpu.TOL["bf16"])
    assert rel_l2(h.cpu().numpy(), h_ref) < 1e-2
    assert torch.all(big[:, :, :1] == 0) and torch.all(big[:, :, 1 + Dn:] == 0)


@pytest.mark.parametrize("batch,heads,headdim,N,groups,L,kw", [
    (2, 5, 32, 64, 1, 1, {}),                        # one tile a workgroup; a width of two and a half tiles; shorter than the conv's reach
    (3, 3, 64, 128, 1, 32, {}),                      # the longest block
    (2, 8, 64, 128, 2, 31, dict(d_conv=3)),          # two groups
    (70, 8, 64, 64, 2, 7, {}),                       # three tiles a workgroup do not make up a group of four: two launches
    (50, 8, 64, 64, 2, 5, {}),                       # two groups, two tiles a workgroup
    (130, 3, 64, 64, 1, 2, {}),                      # two tiles a workgroup, the last of which has one
    (100, 3, 64, 128, 3, 2, {}),                     # groups of one tile, two a workgroup: two launches
    (129, 6, 32, 64, 1, 33, {}),                     # more than 32 tokens: two launches
    (100, 5, 64, 128, 1, 9, dict(conv_bc=0)),        # three tiles a workgroup, B and C as they come
    (85, 10, 64, 64, 1, 3, dict(d_conv=2)),          # four tiles, the last workgroup with two; in place: two launches
    (65, 16, 64, 64, 1, 4, dict(dt_softplus=0)),     # more than four tiles each: two launches
])
def test_ssd_block_forms_agree(gpu, oracle, batch, heads, headdim, N, groups, L, kw):
    """Block calls of every number of tiles a workgroup and those that take two launches, from a cached state and tail and from
    nothing, with the state committed, the tail committed to a buffer of its own and in place, and neither."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.m2_cfg(batch, L, heads * headdim, headdim=headdim, d_state=N, n_groups=groups, **kw)
    pf, pb, inp = case(cfg, 4100 + L + N)
    g = torch.Generator().manual_seed(L + heads)
    K, Dn = cfg["d_conv"], cfg["d_inner"]
    h0 = (0.2 * torch.randn(batch, Dn, N, generator=g)).float()
    tail0 = synth.round_io(torch.randn(batch, K - 1, synth.conv_channels(cfg), generator=g), "bf16")
    sel = sorted({0, headdim - 1, Dn // 2, Dn - 1} | set(np.random.default_rng(L).choice(Dn, size=12, replace=False).tolist()))
    inp_b = synth.make_inputs(cfg, 4200 + L)
    for combine, other, cached in ((0, None, True), (1, inp_b, True), (0, None, False)):
        c = dict(cfg, combine=combine)
        ref, h_ref, t_ref = oracle.bimamba_block_fwd(c, to_np(pf), to_np(pb), to_np(inp), None if other is None else to_np(other),
                                                     h_in=h0.numpy() if cached else None, tail_in=tail0.numpy() if cached else None, sel=sel)
        args = dict(h_in=h0 if cached else None, tail_in=tail0 if cached else None)
        out, h, tail = gpu.gpu_block_fwd(c, pf, pb, inp, other, **args)
        assert_close(out[..., sel], ref, gpu.TOL["bf16"], (combine, cached))
        assert rel_l2(h[:, sel, :], h_ref[:, sel, :]) < 1e-2
        assert np.array_equal(tail, t_ref)
        plain, _, _ = gpu.gpu_block_fwd(c, pf, pb, inp, other, commit=False, **args)
        assert_close(plain[..., sel], ref, gpu.TOL["bf16"], (combine, cached))
        if not cached:
            continue
        desc = bd.make_desc(c)
        dpf, dpb, dinp = bd.to_device(pf), bd.to_device(pb), bd.to_device(inp, c)
        dinp_b = None if other is None else bd.to_device(other, c)
        state, kept = h0.cuda(), tail0.cuda().to(torch.bfloat16)
        res, ws = bd.alloc_out(c), bd.alloc_workspace(desc, 1)
        bd.bimamba_block_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp),
                             None if dinp_b is None else bd.make_inputs(dinp_b), state, kept, state, kept, bd.make_tensor(res), ws)
        torch.cuda.synchronize()
        assert_close(res.float().cpu().numpy().astype(np.float64).reshape(out.shape)[..., sel], ref, gpu.TOL["bf16"], (combine, "in place"))
        assert rel_l2(state.cpu().numpy()[:, sel, :], h_ref[:, sel, :]) < 1e-2
        assert np.array_equal(kept.float().cpu().numpy(), t_ref)


@pytest.mark.parametrize("L,batch,heads,headdim,N,kw", [
    (65, 2, 4, 32, 64, {}),                     # two chunks; the reverse direction's first one holds one token
    (128, 1, 8, 32, 128, {}),                   # two whole chunks
    (66, 1, 3, 32, 64, dict(conv_bc=0)),        # its second chunk's conv window begins before the sequence
    (129, 3, 5, 32, 64, dict(d_conv=3)),        # three chunks: halves of two and one
    (193, 2, 2, 64, 128, {}),                   # four, heads of 64 channels
    (319, 1, 6, 64, 64, dict(n_groups=2)),      # five
    (1111, 1, 3, 64, 128, dict(dt_softplus=0)), # eighteen
    (190, 1, 120, 32, 128, {}),                 # the most heads of 32 channels that the 1.3B layer has
    (250, 2, 64, 64, 64, {}),                   # as many items as there may be
    (129, 1, 4, 64, 64, {}),                    # three chunks, heads of 64 channels: one direction after the other
    (1601, 1, 4, 32, 64, {}),                   # so few items that three time parts are taken instead
])
def test_ssd_directions_meet_in_the_middle(gpu, oracle, L, batch, heads, headdim, N, kw):
    """Directions that are added, few (batch, head) items: gated once and gated each, from nothing and, as a block call, from a cached
    state and tail, with both committed in place."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.m2_cfg(batch, L, heads * headdim, headdim=headdim, d_state=N, **kw)
    pf, pb, inp = case(cfg, 5100 + L + N)
    Dn, K = cfg["d_inner"], cfg["d_conv"]
    g = torch.Generator().manual_seed(L)
    h0 = (0.2 * torch.randn(batch, Dn, N, generator=g)).float()
    tail0 = synth.round_io(torch.randn(batch, K - 1, synth.conv_channels(cfg), generator=g), "bf16")
    sel = sorted({0, headdim - 1, Dn // 2, Dn - 1} | set(np.random.default_rng(L).choice(Dn, size=24, replace=False).tolist()))
    for other in (None, dict(inp, z=synth.make_inputs(cfg, 5300 + L)["z"])):
        both = (to_np(pf), to_np(pb), to_np(inp), None if other is None else to_np(other))
        assert_close(gpu.gpu_fwd(cfg, pf, pb, inp, other)[..., sel], oracle.bimamba_fwd(cfg, *both, sel=sel), gpu.TOL["bf16"], other is None)
        ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, *both, h_in=h0.numpy(), tail_in=tail0.numpy(), sel=sel)
        desc = bd.make_desc(cfg)
        dpf, dpb, dinp = bd.to_device(pf), bd.to_device(pb), bd.to_device(inp, cfg)
        dother = None if other is None else bd.to_device(other, cfg)
        state, kept, res, ws = h0.cuda(), tail0.cuda().to(torch.bfloat16), bd.alloc_out(cfg), bd.alloc_workspace(desc, 1)
        ws.fill_(255)   # (NaN, if anything is read that the call has not written)
        bd.bimamba_block_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp),
                             None if dother is None else bd.make_inputs(dother), state, kept, state, kept, bd.make_tensor(res), ws)
        torch.cuda.synchronize()
        assert_close(res.float().cpu().numpy().astype(np.float64)[..., sel], ref, gpu.TOL["bf16"], (other is None, "block"))
        assert rel_l2(state.cpu().numpy()[:, sel, :], h_ref[:, sel, :]) < 1e-2
        assert np.array_equal(kept.float().cpu().numpy(), t_ref)
