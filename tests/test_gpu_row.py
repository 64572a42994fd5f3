"""GPU parity of the one-launch form of short calls with few chains (a row of 16 lanes per chain): lengths around its groups
of 16 tokens and its time segments, state counts below the row's width, ragged channel tiles, both entry points."""
import numpy as np
import pytest
import torch

from helpers import assert_close, rel_l2, to_np
from paper_2511_15927_amd import synth
from test_gpu_block import params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import gpu_util
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return gpu_util


@pytest.mark.parametrize("L", [1, 2, 15, 16, 17, 31, 33, 48, 64, 65, 100, 127, 129, 200, 255, 256])
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_lengths(gpu, oracle, L, io):
    """Full-sequence and block calls over both dtypes, every conv width, shared and separate activations."""
    k = L % 4
    cfg = synth.mixer_cfg(2, L, (72, 3, 130, 257)[k], d_state=(16, 8, 4, 16)[k], d_conv=1 + (L // 2) % 4, io=io,
                          dt_softplus=L % 2, combine=(L // 3) % 2)
    pf, pb = params(cfg, L, random_a=bool(L & 4))
    inp = synth.make_inputs(cfg, L)
    inp_b = synth.make_inputs(cfg, L + 500) if L % 3 == 0 else None
    both = (to_np(pf), to_np(pb), to_np(inp), None if inp_b is None else to_np(inp_b))
    assert_close(gpu.gpu_fwd(cfg, pf, pb, inp, inp_b), oracle.bimamba_fwd(cfg, *both), gpu.TOL[io])
    g = torch.Generator().manual_seed(L)
    h0 = (0.2 * torch.randn(2, cfg["d_inner"], cfg["d_state"], generator=g)).float()
    K = cfg["d_conv"]
    tail0 = synth.round_io(torch.randn(2, K - 1, cfg["d_inner"], generator=g), io) if K > 1 else None
    ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, *both, h_in=h0.numpy(), tail_in=None if tail0 is None else tail0.numpy())
    got, h_got, t_got = gpu.gpu_block_fwd(cfg, pf, pb, inp, inp_b, h_in=h0, tail_in=tail0)
    assert_close(got, ref, gpu.TOL[io])
    assert rel_l2(h_got, h_ref) < 1e-5
    if K > 1:
        assert np.array_equal(t_got, t_ref)


@pytest.mark.parametrize("L", [31, 128])
def test_heads_groups_and_scalar_decay(gpu, oracle, L):
    """Heads of several channels, two B/C groups, a scalar decay and a skip weight per head."""
    for a_kind in (0, 1):
        cfg = synth.mixer_cfg(1, L, 256, d_state=16, n_heads=32, n_groups=2, a_kind=a_kind, d_kind=1, io="f32")
        pf, pb = synth.make_params(cfg, L, 0), synth.make_params(cfg, L, 1)
        inp = synth.make_inputs(cfg, L)
        assert_close(gpu.gpu_fwd(cfg, pf, pb, inp), oracle.bimamba_fwd(cfg, to_np(pf), to_np(pb), to_np(inp)), gpu.TOL["f32"])


@pytest.mark.parametrize("batch,L,Dn,N,K", [
    (1, 31, 2050, 16, 4),        # two tiles of four channels in a workgroup
    (3, 16, 1366, 8, 3),         # four, a ragged last workgroup of six channels
    (1, 32, 4100, 16, 4),        # four, a last workgroup of one tile
    (2, 64, 2045, 16, 2),        # four, two time segments
    (1, 100, 3001, 4, 4),        # two, two segments
    (1, 128, 2046, 16, 4),       # two, four segments
    (2, 17, 8000, 16, 1),        # four
    (2, 33, 8000, 16, 4),        # four, added up; halves apart: two lanes per chain, not this form
    (2, 17, 6144, 8, 4),         # four, added up; halves apart: one lane per chain
    (1, 50, 33000, 16, 4)])      # not this form: one lane per chain added up, two lanes with the halves apart
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_several_channel_tiles_in_a_workgroup(gpu, oracle, batch, L, Dn, N, K, io):
    """Calls of 2048 chains or more put two or four channel tiles into a workgroup: full-sequence calls with the directions
    added and kept apart, shared and separate activations, and a block call committed in place."""
    from paper_2511_15927_amd import binding as bd
    assert bd.bimamba_time_chunks(bd.make_desc(synth.mixer_cfg(batch, L, Dn, d_state=N))) == 1
    for combine in (0, 1):
        cfg = synth.mixer_cfg(batch, L, Dn, d_state=N, d_conv=K, io=io, dt_softplus=combine, combine=combine)
        pf, pb = params(cfg, Dn + combine, random_a=bool(combine))
        inp = synth.make_inputs(cfg, Dn)
        inp_b = synth.make_inputs(cfg, Dn + 500) if combine else None
        both = (to_np(pf), to_np(pb), to_np(inp), None if inp_b is None else to_np(inp_b))
        assert_close(gpu.gpu_fwd(cfg, pf, pb, inp, inp_b), oracle.bimamba_fwd(cfg, *both), gpu.TOL[io])
        g = torch.Generator().manual_seed(L)
        h0 = (0.2 * torch.randn(batch, Dn, N, generator=g)).float()
        tail0 = synth.round_io(torch.randn(batch, K - 1, Dn, generator=g), io) if K > 1 else None
        ref, h_ref, t_ref = oracle.bimamba_block_fwd(cfg, *both, h_in=h0.numpy(), tail_in=None if tail0 is None else tail0.numpy())
        desc, out, ws = bd.make_desc(cfg), bd.alloc_out(cfg), bd.alloc_workspace(bd.make_desc(cfg), 1)
        dh, dt = h0.cuda(), None if tail0 is None else tail0.to(device="cuda", dtype=bd.io_dtype(cfg))
        dpf, dpb, dinp = bd.to_device(pf), bd.to_device(pb), bd.to_device(inp, cfg)
        dinp_b = None if inp_b is None else bd.to_device(inp_b, cfg)
        bd.bimamba_block_fwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dinp),
                             None if dinp_b is None else bd.make_inputs(dinp_b), dh, dt, dh, dt, bd.make_tensor(out), ws)
        torch.cuda.synchronize()
        assert_close(out.float().cpu().numpy().reshape(ref.shape), ref, gpu.TOL[io])
        assert rel_l2(dh.cpu().numpy(), h_ref) < 1e-5
        if K > 1:
            assert np.array_equal(dt.float().cpu().numpy().astype(np.float64), t_ref)


@pytest.mark.parametrize("batch,L,Dn,N,combine", [
    (13, 16, 1024, 16, 0), (13, 31, 1024, 16, 1), (13, 48, 1024, 16, 1), (9, 16, 1024, 8, 0), (12, 64, 1024, 8, 1), (9, 33, 1024, 4, 0),
])
def test_sizes_of_the_row_form_round_no_decay_more_than_it_does(gpu, oracle, batch, L, Dn, N, combine):
    """Short calls with few chains that another form runs: with an arithmetic A the committed state is as close to 64 bits as with one
    that is a last place away from arithmetic, whose decays are an exponential each whatever the form.  (13 percent: the scatter
    of the norm of 5e4 errors or more is below 1 percent, the two A's own decays differ in their rounding.)"""
    cfg = synth.mixer_cfg(batch, L, Dn, d_state=N, combine=combine)
    pf, pb = synth.make_params(cfg, L, 0), synth.make_params(cfg, L, 1)
    inp = synth.make_inputs(cfg, L)
    error = []
    for last_place in (False, True):
        if last_place:
            for p in (pf, pb):
                p["A"][:, 2] = torch.nextafter(p["A"][:, 2], torch.zeros(()))
        _, h_ref, _ = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp))
        _, h_got, _ = gpu.gpu_block_fwd(cfg, pf, pb, inp)
        error.append(np.linalg.norm(h_got - h_ref) / np.linalg.norm(h_ref))
    assert error[0] < 1.13 * error[1], error


@pytest.mark.parametrize("batch,L,Dn,combine", [(20, 16, 1024, 0), (20, 33, 1024, 1), (25, 64, 1600, 0)])
def test_wide_short_calls_round_no_decay_more_than_lane_pairs_do(gpu, oracle, batch, L, Dn, combine):
    """Short calls of 16 states where lane pairs are the other choice: the committed state is as close to 64 bits as theirs (2 percent: the
    decays are the same bits, only the sum of a token's outputs differs)."""
    cfg = synth.mixer_cfg(batch, L, Dn, combine=combine)
    pf, pb = synth.make_params(cfg, L, 0), synth.make_params(cfg, L, 1)
    inp = synth.make_inputs(cfg, L)
    _, h_ref, _ = oracle.bimamba_block_fwd(cfg, to_np(pf), to_np(pb), to_np(inp))
    error = []
    for split in (0, 2):
        _, h_got, _ = gpu.gpu_block_fwd(dict(cfg, state_split=split), pf, pb, inp)
        error.append(np.linalg.norm(h_got - h_ref) / np.linalg.norm(h_ref))
    assert error[0] < 1.02 * error[1], error
