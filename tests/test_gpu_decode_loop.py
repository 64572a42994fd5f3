"""The block-diffusion decode loop (Sec. 4.3): n_layers x n_steps block calls per block, captured once as a HIP graph
and replayed per block.  Every layer call of every step is checked against the fp64 oracle fed that call's own input
(layer by layer), the committed caches against the oracle's chain, and graph replays against eager runs bit for bit
(several replays, with eager work and synchronisation between them).  Blocks of few chains are one launch (bimamba_block_stack),
which needs no workspace; the same blocks are run call by call too."""
import numpy as np
import pytest
import torch

from helpers import assert_close, rel_l2, to_np
from paper_2511_15927_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout,G,static", [("selective", 32, False), ("selective", 64, True), ("selective_calls", 32, False), ("selective_calls", 64, True),
                                             ("selective_sweep", 32, False), ("selective_sweep", 96, True), ("mamba2", 32, False), ("mamba2", 128, False)])
def test_decode_loop_graph_matches_oracle_layer_by_layer(oracle, layout, G, static):
    from paper_2511_15927_amd import binding as bd
    from paper_2511_15927_amd.decode import BlockDecodeLoop
    assert torch.cuda.is_available(), "these tests need the MI355X"
    n_layers, n_steps, n_blocks = 3, 2, 3
    if layout == "mamba2":
        cfg, h_tol = synth.m2_cfg(2, G, 128, headdim=32, d_state=64), 1e-2
    else:
        cfg, h_tol = synth.mixer_cfg(2, G, 192, time_chunks=int(layout == "selective_sweep")), 1e-5
    Bt, Dn, N, K = cfg["batch"], cfg["d_inner"], cfg["d_state"], cfg["d_conv"]
    params = [(synth.make_params(cfg, 3000 + l, 0), synth.make_params(cfg, 3000 + l, 1)) for l in range(n_layers)]
    loop = BlockDecodeLoop(cfg, params, n_steps, keep_layer_outputs=True, static_scratch=static)
    assert loop._one_launch == (layout in ("selective", "selective_calls"))
    if layout == "selective_calls":
        loop._one_launch = False
    g = torch.Generator().manual_seed(G)
    h_ref, tail_ref = [], []
    for l in range(n_layers):        # a cache as some earlier blocks might have left it
        h0 = (0.2 * torch.randn(Bt, Dn, N, generator=g)).float()
        t0 = synth.round_io(torch.randn(Bt, K - 1, synth.conv_channels(cfg), generator=g), cfg["io"])
        loop.h[l].copy_(h0)
        loop.tail[l].copy_(t0)
        h_ref.append(h0.numpy().astype(np.float64))
        tail_ref.append(t0.numpy().astype(np.float64))
    loop.capture()
    for blk in range(n_blocks):
        steps = [synth.make_inputs(cfg, 3100 + 10 * blk + s) for s in range(n_steps)]
        for s in range(n_steps):
            loop.set_step_inputs(s, steps[s])
        saved = [(h.clone(), t.clone()) for h, t in zip(loop.h, loop.tail)]
        torch.cuda.synchronize()
        loop.run_block()
        torch.cuda.synchronize()
        got = [[loop.layer_output(s, l).float().cpu().numpy() for l in range(n_layers)] for s in range(n_steps)]
        cache = [(h.clone(), t.clone()) for h, t in zip(loop.h, loop.tail)]
        # the same block, eagerly, from the same cache: bit-identical outputs and caches
        for (h0, t0), h, t in zip(saved, loop.h, loop.tail):
            h.copy_(h0)
            t.copy_(t0)
        loop.run_block_eager()
        torch.cuda.synchronize()
        for s in range(n_steps):
            for l in range(n_layers):
                assert np.array_equal(got[s][l], loop.layer_output(s, l).float().cpu().numpy()), (blk, s, l)
        for (h1, t1), h, t in zip(cache, loop.h, loop.tail):
            assert torch.equal(h1, h) and torch.equal(t1, t), blk
        # the oracle, layer by layer, fed each call's own input
        for s in range(n_steps):
            for l in range(n_layers):
                x_in = steps[s]["x"].numpy() if l == 0 else got[s][l - 1]
                ins = dict(to_np(steps[s]), x=x_in)
                ref, h_new, t_new = oracle.bimamba_block_fwd(cfg, to_np(params[l][0]), to_np(params[l][1]), ins,
                                                             h_in=h_ref[l], tail_in=tail_ref[l])
                assert_close(got[s][l], ref, 2e-2, (blk, s, l))
                if s == n_steps - 1:
                    h_ref[l], tail_ref[l] = h_new, t_new
        for l in range(n_layers):
            assert rel_l2(loop.h[l].cpu().numpy(), h_ref[l]) < h_tol, (blk, l)
            assert np.array_equal(loop.tail[l].float().cpu().numpy().astype(np.float64), tail_ref[l]), (blk, l)


def test_decode_loop_prefill_then_blocks_equals_full_forward_scan(oracle):
    """One layer: a prefix scanned once, then committed blocks; the final cached state equals the oracle's forward
    scan of prefix || committed blocks (the block-cache statement of Sec. 4.3 through the loop component)."""
    from paper_2511_15927_amd import binding as bd
    from paper_2511_15927_amd.decode import BlockDecodeLoop
    cfg = synth.mixer_cfg(2, 32, 96)
    pf, pb = synth.make_params(cfg, 3300, 0), synth.make_params(cfg, 3300, 1)
    loop = BlockDecodeLoop(cfg, [(pf, pb)], n_steps=4)
    prefix = synth.make_inputs(cfg, 3301, seqlen=77)
    loop.prefill(bd.to_device({k: v.reshape(v.shape[0], v.shape[1], -1) for k, v in prefix.items()}, cfg), 77)
    loop.capture()
    committed = [to_np(prefix)]
    for blk in range(3):
        for s in range(4):
            inp = synth.make_inputs(cfg, 3310 + 10 * blk + s)
            loop.set_step_inputs(s, inp)
        committed.append(to_np(inp))              # the last step's tokens are the ones committed
        loop.run_block()
    torch.cuda.synchronize()
    whole = {k: np.concatenate([c[k] for c in committed], axis=1) for k in ("x", "z", "dt", "B", "C")}
    _, h_full = oracle.one_direction(dict(cfg, seqlen=77 + 3 * 32), to_np(pf), whole, +1)
    assert rel_l2(loop.h[0].cpu().numpy(), h_full) < 1e-5
    assert np.array_equal(loop.tail[0].float().cpu().numpy(), whole["x"][:, -3:])


@pytest.mark.parametrize("batch,G,Dn,N,keep", [(2, 32, 192, 16, True), (1, 37, 260, 8, False), (1, 100, 1030, 4, True)])
def test_block_in_one_launch_equals_its_calls(batch, G, Dn, N, keep):
    """The one launch against the chain of calls that it stands for, from one cache: fp32 I/O, so that nothing is rounded between the
    layers.  Each side is within 1e-5 of the oracle at every layer (the library's fp32 bound); five layers feed each other."""
    from paper_2511_15927_amd.decode import BlockDecodeLoop
    n_layers, n_steps = 5, 3
    cfg = synth.mixer_cfg(batch, G, Dn, d_state=N, io="f32")
    params = [(synth.make_params(cfg, 3400 + l, 0), synth.make_params(cfg, 3400 + l, 1)) for l in range(n_layers)]
    inputs = [synth.make_inputs(cfg, 3450 + s) for s in range(n_steps)]
    results = []
    for one_launch in (True, False):
        loop = BlockDecodeLoop(cfg, params, n_steps, keep_layer_outputs=keep)
        assert loop._one_launch
        loop._one_launch = one_launch
        g = torch.Generator().manual_seed(G)
        for h, t in zip(loop.h, loop.tail):
            h.copy_(0.2 * torch.randn(h.shape, generator=g))
            t.copy_(torch.randn(t.shape, generator=g))
        for s in range(n_steps):
            loop.set_step_inputs(s, inputs[s])
        loop.run_block_eager()
        torch.cuda.synchronize()
        outs = [loop.layer_output(s, l) for s in range(n_steps) for l in range(n_layers)] if keep else loop.out
        results.append(([t.cpu().numpy() for t in outs + loop.h], [t.cpu() for t in loop.tail]))
    (a, tails_a), (b, tails_b) = results
    for i, (x, y) in enumerate(zip(a, b)):
        assert rel_l2(x, y) < 1e-5 * 2 * n_layers, i
    assert torch.equal(tails_a[0], tails_b[0])                          # the first layer's x is the same
    for x, y in zip(tails_a[1:], tails_b[1:]):
        assert rel_l2(x.numpy(), y.numpy()) < 1e-5 * 2 * n_layers


def test_block_in_a_callers_own_graph():
    """run_block_eager captured without a run before, and again after a step's tensor was replaced: the replays of either graph are the block
    of the tensors that stood there at its capture, whatever ran between."""
    from paper_2511_15927_amd.decode import BlockDecodeLoop
    cfg = synth.mixer_cfg(2, 32, 192)
    params = [(synth.make_params(cfg, 3500 + l, 0), synth.make_params(cfg, 3500 + l, 1)) for l in range(3)]
    loop = BlockDecodeLoop(cfg, params, 2)
    assert loop._one_launch
    for s in range(2):
        loop.set_step_inputs(s, synth.make_inputs(cfg, 3550 + s))
    h0 = [torch.full_like(h, 0.1) for h in loop.h]
    t0 = [torch.zeros_like(t) for t in loop.tail]

    def run(fn):
        for old, new in ((loop.h, h0), (loop.tail, t0)):
            for a, b in zip(old, new):
                a.copy_(b)
        fn()
        torch.cuda.synchronize()
        return [t.clone() for t in loop.out + loop.h + loop.tail]

    def capture():
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            loop.run_block_eager()
        return graph

    same = lambda a, b: all(torch.equal(x, y) for x, y in zip(a, b))
    old_x = loop.step_inputs[0]["x"]
    first = capture()
    want_first = run(loop.run_block_eager)
    assert same(run(first.replay), want_first)
    loop.step_inputs[0]["x"] = torch.ones_like(old_x)
    second = capture()                       # (call by call)
    want_second = run(loop.run_block_eager)  # (uploads the table anew)
    loop._one_launch = False
    want_calls = run(loop.run_block_eager)
    loop._one_launch = True
    for _ in range(3):
        assert same(run(first.replay), want_first)
        assert same(run(second.replay), want_calls)
        assert same(run(loop.run_block_eager), want_second)
    assert not torch.equal(want_first[0], want_second[0])


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("batch,L,Dn,kw", [
    (1, 1, 5, dict(d_state=4)),                                  # rows shorter than a piece of eight
    (3, 7, 8, dict(d_state=8)),                                  # one piece each
    (2, 33, 130, {}),                                            # a remainder of two
    (1, 32, 4096, {}),                                           # several workgroups
    (2, 5, 192, dict(n_heads=24, n_groups=3, d_state=8)),        # B and C of three groups, few dt columns
])
def test_copy_inputs_rows_at_any_place(io, batch, L, Dn, kw):
    """bimamba_copy_inputs bit for bit, between contiguous tensors and column slices at 16-byte and at odd places on either side, batch strides
    of their own; what lies around the places stays."""
    from paper_2511_15927_amd import binding as bd
    cfg = synth.mixer_cfg(batch, L, Dn, io=io, **kw)
    desc, dtype, GN = bd.make_desc(cfg), bd.io_dtype(cfg), cfg["n_groups"] * cfg["d_state"]
    widths = dict(x=Dn, z=Dn, dt=cfg["n_heads"], B=GN, C=GN)
    g = torch.Generator(device="cuda").manual_seed(L + Dn)

    def sides(pad, at):      # one buffer a tensor: `at` columns in front, so many in all that rows are `pad` apart modulo 8, a batch element to spare
        whole = {k: torch.randn(batch, L + 1, (n + at + 7) // 8 * 8 + pad, device="cuda", generator=g).to(dtype) for k, n in widths.items()}
        return whole, {k: w[:, :L, at:at + widths[k]] for k, w in whole.items()}

    plain = {k: torch.randn(batch, L, n, device="cuda", generator=g).to(dtype) for k, n in widths.items()}
    for src in (plain, sides(0, 8)[1], sides(8, 0)[1], sides(3, 1)[1]):
        for pad, at in ((0, 0), (8, 16), (0, 1), (5, 2)):
            whole, dst = sides(pad, at)
            kept = {k: w.clone() for k, w in whole.items()}
            for k, n in widths.items():
                kept[k][:, :L, at:at + n] = src[k]
            four = {k: v if k in "xz" or k == "dt" else v.unflatten(2, (cfg["n_groups"], -1)) for k, v in src.items()}
            bd.bimamba_copy_inputs(desc, bd.make_inputs(four), bd.make_inputs(dst))
            torch.cuda.synchronize()
            for k in widths:
                assert torch.equal(whole[k], kept[k]), (k, pad, at)


@pytest.mark.parametrize("kind,at_once", [("same", 1), ("columns", 1), ("odd columns", 1), ("transposed", 1), ("flat rows", 1), ("groups apart", 1), ("one row", 1),
                                          ("parameter", 1), ("own", 0), ("own, turned", 0), ("other dtype", 0), ("host", 0), ("grad", 0), ("replaced", 0), ("moved", 0)])
def test_step_inputs_refreshed_in_one_launch(kind, at_once, monkeypatch):
    """set_step_inputs with tensors on the device: the values asked for, in one launch of the library where they are of the buffer's kind, and
    the other step as it was."""
    from paper_2511_15927_amd import binding as bd
    from paper_2511_15927_amd.decode import BlockDecodeLoop
    cfg = synth.mixer_cfg(2, 9, 128, n_groups=2, n_heads=16, d_state=4)
    loop = BlockDecodeLoop(cfg, [(synth.make_params(cfg, 1, 0), synth.make_params(cfg, 1, 1))], 2)
    real, statuses = bd.bimamba_copy_inputs, []

    def counted(*a, **kw):
        statuses.append(real(*a, **kw))
        return statuses[-1]
    monkeypatch.setattr(bd, "bimamba_copy_inputs", counted)
    want = {k: v.to("cuda", torch.bfloat16).reshape(2, 9, -1) for k, v in synth.make_inputs(cfg, 3).items()}
    given = dict(want)
    if kind in ("columns", "odd columns"):
        at = 8 if kind == "columns" else 3
        wide = torch.randn(2, 9, 128 + 128 + 16 + 8 + 8 + at, device="cuda").to(torch.bfloat16)
        for k in given:
            n = want[k].shape[2]
            wide[:, :, at:at + n] = want[k]
            given[k] = wide[:, :, at:at + n]
            at += n
    elif kind == "transposed":
        given["x"] = want["x"].transpose(0, 1).contiguous().transpose(0, 1)
        given["z"] = want["z"].transpose(1, 2).contiguous().transpose(1, 2)
    elif kind == "flat rows":
        given["dt"] = torch.cat([want["dt"], want["dt"]], dim=2).reshape(18, 32)[:, :16]
    elif kind == "groups apart":
        given["B"] = torch.stack([want["B"].unflatten(2, (2, 4))] * 2, dim=3)[:, :, :, 1]
        given["C"] = want["C"].unflatten(2, (2, 4))
    elif kind == "one row":
        want["dt"] = want["dt"][:1, :1].expand(2, 9, 16)
        given["dt"] = want["dt"]
    elif kind == "parameter":
        given["x"] = torch.nn.Parameter(want["x"], requires_grad=False)
    elif kind == "own":
        loop.set_step_inputs(0, dict(want, x=want["z"]))
        given["z"] = loop.step_inputs[0]["x"]       # (read after x has been written)
        want["z"] = want["x"]
    elif kind == "own, turned":      # 128 rows of nine of the buffer of x, which hold the new x by then
        given["z"] = loop.step_inputs[0]["x"].flatten(1).unflatten(1, (128, 9)).transpose(1, 2)
        want["z"] = want["x"].flatten(1).unflatten(1, (128, 9)).transpose(1, 2)
    elif kind == "other dtype":
        given["z"] = want["z"].float()
    elif kind == "host":
        given["z"] = want["z"].cpu()
    elif kind == "grad":
        given["dt"] = want["dt"].clone().requires_grad_()
    elif kind == "replaced":
        loop.step_inputs[0]["x"] = torch.zeros_like(loop.step_inputs[0]["x"])
    elif kind == "moved":
        loop.step_inputs[0]["x"].data = torch.zeros_like(loop.step_inputs[0]["x"])
    statuses.clear()
    version = loop._step_flat[0]._version
    with torch.no_grad():
        loop.set_step_inputs(0, given)
    torch.cuda.synchronize()
    for k, v in want.items():
        assert torch.equal(loop.step_inputs[0][k], v), k
    assert all(t.count_nonzero() == 0 for t in loop.step_inputs[1].values())
    assert statuses.count(0) == at_once and loop._step_flat[0]._version > version
