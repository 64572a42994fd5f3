"""GPU parity of the state-carrying block variant (Sec. 4.3) against the fp64 oracle."""
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


def params(cfg, seed, random_a=True):
    pf, pb = synth.make_params(cfg, seed, 0), synth.make_params(cfg, seed, 1)
    if random_a:
        pf["A"], pb["A"] = synth.random_A(cfg, seed), synth.random_A(cfg, seed + 1)
    return pf, pb


def raw_tail(cfg, inp, upto):
    """Last K-1 raw tokens before index `upto` (zeros where the sequence has not started), [Bt, K-1, tail_ch]."""
    K, Bt = cfg["d_conv"], cfg["batch"]
    cols = [inp["x"]]
    if cfg["conv_bc"]:
        cols += [inp["B"].reshape(Bt, inp["B"].shape[1], -1), inp["C"].reshape(Bt, inp["C"].shape[1], -1)]
    raw = torch.cat(cols, dim=2)
    tail = torch.zeros(Bt, K - 1, raw.shape[2])
    take = min(upto, K - 1)
    if take:
        tail[:, K - 1 - take:] = raw[:, upto - take:upto]
    return tail


@pytest.mark.parametrize("variant", ["s_f32", "s_bf16", "m2_f32", "sep"])
def test_block_matches_oracle_with_carried_state(gpu, oracle, variant):
    if variant == "m2_f32":
        cfg = synth.m2_cfg(2, 48, 128, headdim=32, d_state=16, io="f32")
    else:
        cfg = synth.mixer_cfg(2, 48, 100, io="bf16" if variant == "s_bf16" else "f32",
                              combine=1 if variant == "sep" else 0)
    pf, pb = params(cfg, 11)
    inp = synth.make_inputs(cfg, 11)
    m, G = 21, 16                                           # prefix length and block length
    pre = {k: v[:, :m].contiguous() for k, v in inp.items()}
    blk = {k: v[:, m:m + G].contiguous() for k, v in inp.items()}
    _, h_pre = oracle.one_direction(dict(cfg, seqlen=m), to_np(pf), to_np(pre), +1)
    h_in = h_pre.astype(np.float32)                          # the cached state is fp32 on both sides
    tail = raw_tail(cfg, inp, m)
    cb = dict(cfg, seqlen=G)
    ref, h_ref, t_ref = oracle.bimamba_block_fwd(cb, to_np(pf), to_np(pb), to_np(blk), h_in=h_in, tail_in=tail.numpy())
    got, h_got, t_got = gpu.gpu_block_fwd(cb, pf, pb, blk, h_in=h_in, tail_in=tail)
    assert_close(got, ref, gpu.TOL[cfg["io"]])
    assert rel_l2(h_got, h_ref) < 1e-5
    assert np.array_equal(t_got, t_ref)


def test_block_chain_equals_full_forward_scan(gpu, oracle):
    """Chaining committed blocks reproduces the full-sequence forward state; every block's forward half equals the
    full scan's rows and its reverse half the block-local reverse scan."""
    cfg = synth.mixer_cfg(2, 96, 70, io="f32", combine=1)
    pf, pb = params(cfg, 12)
    inp = synth.make_inputs(cfg, 12)
    g_full, h_full = oracle.one_direction(cfg, to_np(pf), to_np(inp), +1)
    h, tail = None, None
    for t0, t1 in ((0, 32), (32, 33), (33, 35), (35, 35), (35, 96)):
        blk = {k: v[:, t0:t1].contiguous() for k, v in inp.items()}
        cb = dict(cfg, seqlen=t1 - t0)
        out, h, tail = gpu.gpu_block_fwd(cb, pf, pb, blk, h_in=h, tail_in=tail)
        if t1 > t0:
            g_rev, _ = oracle.one_direction(cb, to_np(pb), to_np(blk), -1)
            assert rel_l2(out[:, :, 0], g_full[:, t0:t1]) < 1e-5, (t0, t1)
            assert rel_l2(out[:, :, 1], g_rev) < 1e-5, (t0, t1)
    assert rel_l2(h, h_full) < 1e-5
    assert np.array_equal(tail, inp["x"][:, 93:96].numpy().astype(np.float64))


@pytest.mark.parametrize("kw", [{}, dict(state_split=1, time_chunks=1), dict(state_split=2, time_chunks=1)])
def test_block_no_commit_and_in_place_commit(gpu, oracle, kw):
    """On the form the library picks and on those of the sweep: one launch, lanes split."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.mixer_cfg(2, 32, 128, io="bf16", **kw)
    pf, pb = params(cfg, 13)
    inp = synth.make_inputs(cfg, 13)
    h0 = (0.1 * torch.randn(2, 128, 16, generator=torch.Generator().manual_seed(5))).float()
    tail0 = synth.round_io(torch.randn(2, 3, 128, generator=torch.Generator().manual_seed(6)), "bf16")
    ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), h_in=h0.numpy(), tail_in=tail0.numpy())
    # denoising steps that do not commit leave the cache untouched
    got, h_none, t_none = gpu.gpu_block_fwd(cfg, pf, pb, inp, h_in=h0, tail_in=tail0, commit=False)
    assert h_none is None and t_none is None
    assert_close(got, ref, gpu.TOL["bf16"])
    # committing in place (h_out aliases h_in, tail_out aliases tail_in)
    desc = bd.make_desc(cfg)
    dh, dt = h0.cuda(), tail0.to(torch.bfloat16).cuda()
    out = bd.alloc_out(cfg)
    dpf, dpb, dinp, ws = bd.to_device(pf), bd.to_device(pb), bd.to_device(inp, cfg), bd.alloc_workspace(desc, 1)
    bd.bimamba_block_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp), None, dh, dt, dh, dt,
                         bd.make_tensor(out), ws)
    torch.cuda.synchronize()
    assert_close(out.float().cpu().numpy(), ref, gpu.TOL["bf16"])
    assert rel_l2(dh.cpu().numpy(), h_ref) < 1e-5
    assert np.array_equal(dt.float().cpu().numpy().astype(np.float64), t_ref)


@pytest.mark.parametrize("chunks", [2, 5])
def test_block_long_prefix_time_chunked(gpu, oracle, chunks):
    """A long clean prefix scanned once through the block entry point, cut into time segments: the committed state
    must equal the sequential scan's (and may be written in place)."""
    cfg = synth.mixer_cfg(1, 333, 96, io="f32", time_chunks=chunks)
    pf, pb = params(cfg, 14)
    inp = synth.make_inputs(cfg, 14)
    h0 = (0.1 * torch.randn(1, 96, 16, generator=torch.Generator().manual_seed(7))).float()
    ref, h_ref, _ = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), h_in=h0.numpy())
    got, h_got, _ = gpu.gpu_block_fwd(cfg, pf, pb, inp, h_in=h0)
    assert rel_l2(got, ref) < 1e-5
    assert rel_l2(h_got, h_ref) < 1e-5


def test_cfg3_block_diffusion_shapes(gpu, oracle):
    """batch 16, d_inner 4096: a clean prefix scanned once (forward state cached), then 32-token blocks re-scanned
    several denoising steps from the cached state, committing on a block's last step."""
    cfg_p = dict(synth.CONFIGS["cfg3_prefix"], seqlen=1024)       # shortened prefix keeps the test quick
    cfg_b = synth.CONFIGS["cfg3_block"]
    Bt, Dn, N, G = 16, 4096, 16, 32
    seed = synth.config_seed(3)
    pf, pb = params(cfg_p, seed, random_a=False)
    sel = sorted(np.random.default_rng(6).choice(Dn, size=16, replace=False).tolist())
    prefix = synth.make_inputs(cfg_p, seed)
    out_p, h_gpu, tail_gpu = gpu.gpu_block_fwd(cfg_p, pf, pb, prefix)
    ref_p, h_ref, tail_ref = oracle.bimamba_block_fwd(cfg_p, to_np(pf), to_np(pb), to_np(prefix), sel=sel)
    assert_close(out_p[..., sel], ref_p, gpu.TOL["bf16"])
    assert rel_l2(h_gpu[:, sel], h_ref[:, sel]) < 1e-5
    assert np.array_equal(tail_gpu, tail_ref)
    for blk in range(2):
        for step in range(3):
            last = step == 2
            inp = synth.make_inputs(cfg_b, seed + 10 * blk + step + 1)      # the block's tokens change every step
            got, h_new, tail_new = gpu.gpu_block_fwd(cfg_b, pf, pb, inp, h_in=h_gpu, tail_in=tail_gpu, commit=last)
            ref, h_ref_new, tail_ref_new = oracle.bimamba_block_fwd(cfg_b, to_np(pf), to_np(pb), to_np(inp),
                                                                   h_in=h_ref, tail_in=tail_ref, sel=sel)
            assert_close(got[..., sel], ref, gpu.TOL["bf16"], (blk, step))
            if last:
                h_gpu, tail_gpu, h_ref, tail_ref = h_new, tail_new, h_ref_new, tail_ref_new
                assert rel_l2(h_gpu[:, sel], h_ref[:, sel]) < 1e-5
                assert np.array_equal(tail_gpu, tail_ref)


@pytest.mark.parametrize("layout", ["selective", "mamba2"])
def test_empty_sequence_and_empty_batch(gpu, oracle, layout):
    """L = 0: nothing is computed, the cached state and conv tail pass through unchanged (zero state when there is
    none); batch = 0: a no-op.  Both must return without touching memory they were not given."""
    from paper_2511_15927_amd import binding as bd
    if layout == "selective":
        cfg = synth.mixer_cfg(2, 0, 128, io="bf16")
    else:
        cfg = synth.m2_cfg(2, 0, 128, headdim=64, d_state=64)
    pf, pb = params(cfg, 21)
    inp = synth.make_inputs(cfg, 21)
    N, K = cfg["d_state"], cfg["d_conv"]
    tail_ch = 128 + (2 * N if cfg["conv_bc"] else 0)
    h0 = (0.1 * torch.randn(2, 128, N, generator=torch.Generator().manual_seed(7))).float()
    tail0 = synth.round_io(torch.randn(2, K - 1, tail_ch, generator=torch.Generator().manual_seed(8)), "bf16")
    ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), h_in=h0.numpy(), tail_in=tail0.numpy())
    out, h, tail = gpu.gpu_block_fwd(cfg, pf, pb, inp, h_in=h0, tail_in=tail0)
    assert out.shape == ref.shape == (2, 0, 128)
    assert np.array_equal(h, h_ref) and np.array_equal(h, h0.numpy().astype(np.float64))
    assert np.array_equal(tail, t_ref)
    # no cached state: the committed state is zero
    _, h_zero, _ = gpu.gpu_block_fwd(cfg, pf, pb, inp, h_in=None, tail_in=None)
    assert np.array_equal(h_zero, np.zeros_like(h_zero))
    # full-sequence entry point on an empty sequence and on an empty batch
    assert gpu.gpu_fwd(cfg, pf, pb, inp).shape == (2, 0, 128)
    cfg0 = dict(cfg, batch=0, seqlen=5)
    inp0 = synth.make_inputs(cfg0, 22)
    assert gpu.gpu_fwd(cfg0, pf, pb, inp0).shape == (0, 5, 128)
    desc = bd.make_desc(cfg)
    assert bd.bimamba_time_chunks(desc) >= 1


@pytest.mark.parametrize("layout", ["selective", "selective_sweep", "mamba2"])
def test_block_step_replayed_from_a_hip_graph(gpu, layout):
    """One committing block call captured into a HIP graph: every replay (with eager work and synchronisation between
    replays, and fresh contents in the static input buffers) must equal the eager call on the same contents bit for bit."""
    from paper_2511_15927_amd import binding as bd
    if layout == "mamba2":
        cfg = synth.m2_cfg(4, 32, 256, headdim=64, d_state=64)
    else:
        cfg = synth.mixer_cfg(4, 32, 256, io="bf16", time_chunks=int(layout == "selective_sweep"))
    N, K = cfg["d_state"], cfg["d_conv"]
    tail_ch = 256 + (2 * N if cfg["conv_bc"] else 0)
    pf, pb = params(cfg, 31, random_a=False)
    dpf, dpb = bd.to_device(pf), bd.to_device(pb)
    cpf, cpb = bd.make_params(dpf), bd.make_params(dpb)
    desc = bd.make_desc(cfg)
    static_in = bd.to_device(synth.make_inputs(cfg, 31), cfg)
    c_in = bd.make_inputs(static_in)
    h_in = torch.zeros(4, 256, N, dtype=torch.float32, device="cuda")
    tail_in = torch.zeros(4, K - 1, tail_ch, dtype=torch.bfloat16, device="cuda")
    h_out, tail_out = torch.empty_like(h_in), torch.empty_like(tail_in)
    out, ws = bd.alloc_out(cfg), bd.alloc_workspace(desc, 1)
    c_out = bd.make_tensor(out)

    def call():
        bd.bimamba_block_fwd(desc, cpf, cpb, c_in, None, h_in, tail_in, h_out, tail_out, c_out, ws)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for rep in range(3):
        fresh = bd.to_device(synth.make_inputs(cfg, 40 + rep), cfg)
        for k in static_in:
            static_in[k].copy_(fresh[k])
        h_in.copy_(0.1 * torch.randn(4, 256, N, generator=torch.Generator().manual_seed(50 + rep)))
        tail_in.copy_(torch.randn(4, K - 1, tail_ch, generator=torch.Generator().manual_seed(60 + rep)).to(torch.bfloat16))
        call()
        torch.cuda.synchronize()
        want = (out.clone(), h_out.clone(), tail_out.clone())
        out.zero_(); h_out.zero_(); tail_out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[0]) and torch.equal(h_out, want[1]) and torch.equal(tail_out, want[2]), rep


@pytest.mark.parametrize("layout", ["selective", "selective_sweep", "mamba2"])
def test_first_call_in_a_process_captured_into_a_graph(layout):
    """A kernel variant's first launch in a process triggers the library's one-time queries for it; here that first
    launch happens under stream capture (a fresh child process whose first library call is the captured one).  The
    capture must succeed and every replay must match the oracle and an eager call."""
    import json
    import os
    import subprocess
    import sys
    child = os.path.join(os.path.dirname(os.path.abspath(__file__)), "capture_first_use_child.py")
    r = subprocess.run([sys.executable, child, layout], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    res = json.loads(r.stdout.strip().splitlines()[-1])
    assert res["eager_equals_replay"], res
    for rep in res["replays"]:
        assert rep["out"] < 2e-2 and rep["h"] < (1e-2 if layout == "mamba2" else 1e-5) and rep["tail_equal"], res


@pytest.mark.parametrize("L", [1, 2, 3, 7, 41])
@pytest.mark.parametrize("split,N,K,io", [(1, 16, 4, "bf16"), (1, 16, 3, "f32"), (1, 16, 2, "bf16"), (1, 8, 4, "f32"), (1, 8, 3, "bf16"),
                                          (1, 4, 2, "f32"), (1, 4, 4, "bf16"),      # the short form: dtypes, conv widths, states
                                          (2, 16, 3, "bf16"), (4, 16, 4, "f32"), (1, 32, 2, "f32"), (4, 64, 4, "bf16")])
def test_tail_committed_by_the_sweep(gpu, oracle, L, split, N, K, io):
    """The short form of the sweep (one lane per chain, up to 16 states) stores the conv tail itself: calls shorter and longer
    than the tail, with and without one to start from, an odd number of channel tiles, the halves added and kept apart,
    committed in place; other forms and calls cut into segments leave the tail to its own launch."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.mixer_cfg(2, L, 64 + 3 * (64 // split) // 2, d_state=N, d_conv=K, io=io, combine=L % 2)
    pf, pb = params(cfg, 77 + L)
    inp = synth.make_inputs(cfg, 78 + L)
    g = torch.Generator().manual_seed(79 + L)
    h0 = (0.2 * torch.randn(2, cfg["d_inner"], N, generator=g)).float()
    tail0 = synth.round_io(torch.randn(2, K - 1, cfg["d_inner"], generator=g), io) if L != 2 else None
    ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), h_in=h0.numpy(),
                                                 tail_in=None if tail0 is None else tail0.numpy())
    for chunks in (1, 2):
        got, h, t = gpu.gpu_block_fwd(cfg, pf, pb, inp, h_in=h0, tail_in=tail0, state_split=split, time_chunks=chunks)
        assert_close(got.reshape(ref.shape), ref, gpu.TOL[io])
        assert rel_l2(h, h_ref) < 1e-5
        assert np.array_equal(t, t_ref)
    if tail0 is None:
        return
    desc = bd.make_desc(cfg, state_split=split, time_chunks=1)
    dh, dt = h0.cuda(), tail0.to(device="cuda", dtype=bd.io_dtype(cfg))
    out = bd.alloc_out(cfg)
    dpf, dpb, dinp, ws = bd.to_device(pf), bd.to_device(pb), bd.to_device(inp, cfg), bd.alloc_workspace(desc, 1)
    bd.bimamba_block_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp), None, dh, dt, dh, dt,
                         bd.make_tensor(out), ws)
    torch.cuda.synchronize()
    assert_close(out.float().cpu().numpy().reshape(ref.shape), ref, gpu.TOL[io])
    assert np.array_equal(dt.float().cpu().numpy().astype(np.float64), t_ref)


@pytest.mark.parametrize("L", [1, 2, 8, 15, 16, 17, 33, 63, 64])
@pytest.mark.parametrize("N,io,a_kind,own", [(16, "bf16", 0, ""), (16, "f32", 0, "z"), (16, "bf16", 1, "BC"), (8, "bf16", 0, "xzBC"), (4, "f32", 1, "BC")])
def test_one_launch_short_calls(gpu, oracle, L, N, io, a_kind, own):
    """Calls of up to 64 tokens, one lane per chain, in one launch: around the tiles of eight tokens and the meeting of the
    directions; B/C groups whose border lies inside a workgroup; the reverse direction with `own` tensors for some of its inputs
    (gated together or apart, one copy of B and C rows or two); general and arithmetic decays, decays per head; halves apart;
    states and tails committed in place."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.mixer_cfg(2, L, 192, d_state=N, n_heads=192 if L % 2 else 96, n_groups=3, io=io, a_kind=a_kind, dt_softplus=L // 2 % 2,
                          combine=int(L in (2, 15, 33)))   # (64 tokens, halves together, two groups and own B, C: the most LDS)
    if a_kind == 0 and L % 4 != 1:
        pf, pb = params(cfg, 60 + L)
    else:
        pf, pb = synth.make_params(cfg, 60 + L, 0), synth.make_params(cfg, 60 + L, 1)
    inp, other = synth.make_inputs(cfg, 61 + L), synth.make_inputs(cfg, 62 + L)
    inp_b = {k: other[k] if k in own else v for k, v in inp.items()}
    g = torch.Generator().manual_seed(63 + L)
    h0 = (0.2 * torch.randn(2, 192, N, generator=g)).float()
    tail0 = synth.round_io(torch.randn(2, 3, 192, generator=g), io)
    ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), to_np(inp_b), h_in=h0.numpy(), tail_in=tail0.numpy())
    desc = bd.make_desc(cfg, state_split=1, time_chunks=1)
    dev_f, dev_o = bd.to_device(inp, cfg), bd.to_device(other, cfg)
    dev_b = {k: dev_o[k] if k in own else v for k, v in dev_f.items()}
    dh, dt = h0.cuda(), tail0.to(device="cuda", dtype=bd.io_dtype(cfg))
    out, dpf, dpb, ws = bd.alloc_out(cfg), bd.to_device(pf), bd.to_device(pb), bd.alloc_workspace(desc, 1)
    bd.bimamba_block_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dev_f), bd.make_inputs(dev_b), dh, dt, dh, dt,
                         bd.make_tensor(out), ws)
    torch.cuda.synchronize()
    assert_close(out.float().cpu().numpy().reshape(ref.shape), ref, gpu.TOL[io])
    assert rel_l2(dh.cpu().numpy(), h_ref) < 1e-5
    assert np.array_equal(dt.float().cpu().numpy().astype(np.float64), t_ref)


@pytest.mark.parametrize("form,cfg", [
    ("row", synth.mixer_cfg(1, 17, 68, io="f32")),
    ("one launch", synth.mixer_cfg(2, 9, 192, state_split=1, time_chunks=1)),
    ("sweep", synth.mixer_cfg(2, 75, 192, time_chunks=1)),
    ("m2, lane per chain", synth.m2_cfg(2, 6, 128, headdim=32, d_state=16)),
    ("m2, one launch", synth.m2_cfg(3, 32, 192, headdim=64, d_state=128)),
    ("m2, one launch, shorter than the tail", synth.m2_cfg(2, 2, 256, headdim=32, d_state=64, n_groups=2)),
    ("m2, one launch, conv of three", synth.m2_cfg(1, 31, 96, headdim=32, d_state=128, d_conv=3)),
    ("m2, one launch, two tiles a workgroup", synth.m2_cfg(50, 5, 512, headdim=64, d_state=64, n_groups=2)),
    ("m2, four tiles a workgroup", synth.m2_cfg(85, 3, 640, headdim=64, d_state=64)),
    ("m2, two launches", synth.m2_cfg(2, 33, 192, headdim=64, d_state=128)),
    ("m2, chunks", synth.m2_cfg(2, 129, 128, headdim=64, d_state=64)),
])
@pytest.mark.parametrize("cached", [True, False])
def test_state_and_tail_are_committed_each_by_itself(gpu, oracle, form, cfg, cached):
    """h_out and tail_out do not depend on each other: either, both or neither, from a cached state and tail and from none, with the
    directions' activations shared and apart; what is committed is written whole (its buffers hold NaN before)."""
    from paper_2511_15927_amd import binding as bd
    pf, pb = synth.make_params(cfg, 70, 0), synth.make_params(cfg, 70, 1)
    inp, inp_b = synth.make_inputs(cfg, 71), synth.make_inputs(cfg, 72)
    Bt, Dn, N, K, ch = cfg["batch"], cfg["d_inner"], cfg["d_state"], cfg["d_conv"], synth.conv_channels(cfg)
    g = torch.Generator().manual_seed(73)
    h0 = (0.2 * torch.randn(Bt, Dn, N, generator=g)).float() if cached else None
    tail0 = synth.round_io(torch.randn(Bt, K - 1, ch, generator=g), cfg["io"]) if cached else None
    desc, dpf, dpb = bd.make_desc(cfg), bd.to_device(pf), bd.to_device(pb)
    dinp, ws = bd.to_device(inp, cfg), bd.alloc_workspace(desc, 1)
    h_tol = 1e-2 if form.startswith("m2") and cfg["d_state"] >= 64 else 1e-5     # (the matrix-core path takes the state from bf16 operands)
    for other in (None, inp_b):
        ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp), None if other is None else to_np(other),
                                                     h_in=None if h0 is None else h0.numpy(), tail_in=None if tail0 is None else tail0.numpy())
        dother = None if other is None else bd.to_device(other, cfg)
        for with_h in (False, True):
            for with_tail in (False, True):
                h = torch.full((Bt, Dn, N), float("nan"), device="cuda") if with_h else None
                tail = torch.full((Bt, K - 1, ch), float("nan"), dtype=bd.io_dtype(cfg), device="cuda") if with_tail else None
                out = bd.alloc_out(cfg)
                bd.bimamba_block_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp),
                                     None if dother is None else bd.make_inputs(dother), None if h0 is None else h0.cuda(),
                                     None if tail0 is None else tail0.to(device="cuda", dtype=bd.io_dtype(cfg)), h, tail, bd.make_tensor(out), ws)
                torch.cuda.synchronize()
                what = (other is not None, with_h, with_tail)
                assert_close(out.float().cpu().numpy(), ref, gpu.TOL[cfg["io"]], what)
                if with_h:
                    assert rel_l2(h.cpu().numpy(), h_ref) < h_tol, what
                if with_tail:
                    assert np.array_equal(tail.float().cpu().numpy().astype(np.float64), t_ref), what
