"""GPU parity of bimamba_bwd (gradients of the full-sequence path, selective-scan layout) against the fp64 oracle's
gradients, which are themselves pinned by finite differences and automatic differentiation (test_oracle_bwd_pins.py).

Tolerances: a gradient tensor is compared in relative L2 over the whole tensor; fp32 I/O 2e-5 (fp32 arithmetic, sums of
up to L * batch terms formed in a fixed order), bf16 I/O 2e-2 for the tensors that are rounded to bf16
(dx, dz, ddt) and 2e-5 for the fp32 ones (dB, dC and the parameter gradients see the same fp32 arithmetic in both modes).
"""
import numpy as np
import pytest
import torch

from helpers import rel_l2, to_np
from paper_2511_15927_amd import binding as bd
from paper_2511_15927_amd import synth
from test_gpu_block import params

pytestmark = pytest.mark.gpu

FP32_TOL, BF16_TOL = 2e-5, 2e-2


@pytest.fixture(scope="module")
def gpu():
    import gpu_util
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return gpu_util


def rounded(a, io):
    t = torch.as_tensor(a, dtype=torch.float32)
    return (t.to(torch.bfloat16).float() if io == "bf16" else t).numpy()


def rel_all(got, ref):
    """Relative L2 over a whole tensor (parameter gradients have no batch dimension to take a maximum over)."""
    return float(np.linalg.norm(np.asarray(got) - np.asarray(ref)) / np.linalg.norm(np.asarray(ref)))


def compare(cfg, got, ref, sel=None):
    io_tol = BF16_TOL if cfg["io"] == "bf16" else FP32_TOL
    gf, gb, qf, qb = got
    rf, rb, pf, pb = ref
    pick = (lambda a: a[..., sel]) if sel is not None else (lambda a: a)
    worst = {}
    for tag, g, r in (("f", gf, rf), ("b", gb, rb)):
        if r is None:
            assert g is None
            continue
        for k in ("dx", "dz"):
            worst[tag + k] = rel_l2(pick(g[k]), r[k])
            assert worst[tag + k] < io_tol, (tag, k, worst)
        worst[tag + "ddt"] = rel_l2(pick(g["ddt"]), pick(r["ddt"]))
        assert worst[tag + "ddt"] < io_tol, (tag, "ddt", worst)
        if sel is None:
            for k in ("dB", "dC"):
                worst[tag + k] = rel_l2(g[k], r[k])
                assert worst[tag + k] < FP32_TOL, (tag, k, worst)
    for tag, g, r in (("f", qf, pf), ("b", qb, pb)):
        for k in ("dconv_w", "dconv_b", "dA", "dD", "ddt_bias"):
            a, b = (g[k][sel], r[k][sel]) if sel is not None else (g[k], r[k])
            if not np.any(b):
                assert not np.any(a), (tag, k)
                continue
            worst[tag + k] = rel_all(a, b)
            assert worst[tag + k] < FP32_TOL, (tag, k, worst)
    return worst


def run_case(gpu, oracle, cfg, seed, untied=False, random_a=True):
    pf, pb = params(cfg, seed, random_a=random_a)
    in_f = synth.make_inputs(cfg, seed)
    in_b = synth.make_inputs(cfg, seed + 500) if untied else None
    width = cfg["d_inner"] * (2 if cfg["combine"] else 1)
    g = torch.Generator().manual_seed(seed + 9)
    dout = rounded(torch.randn(cfg["batch"], cfg["seqlen"], width, generator=g), cfg["io"])
    got = gpu.gpu_bwd(cfg, pf, pb, in_f, in_b, dout)
    ref = oracle.bimamba_bwd(cfg, to_np(pf), to_np(pb), to_np(in_f), None if in_b is None else to_np(in_b), dout)
    return compare(cfg, got, ref)


@pytest.mark.parametrize("L", [1, 2, 7, 8, 9, 16, 23, 100])
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_lengths_around_the_chunks(gpu, oracle, L, io):
    run_case(gpu, oracle, synth.mixer_cfg(2, L, 72, io=io), 10 + L)


@pytest.mark.parametrize("N", [4, 8, 16])
@pytest.mark.parametrize("K", [1, 2, 3, 4])
def test_state_sizes_and_conv_widths(gpu, oracle, N, K):
    run_case(gpu, oracle, synth.mixer_cfg(2, 37, 130, d_state=N, d_conv=K, io="f32"), 30 + N + K)


@pytest.mark.parametrize("mode", ["separate", "untied", "untied_separate", "softplus", "groups", "progression_a"])
def test_modes(gpu, oracle, mode):
    kw = {}
    if "separate" in mode:
        kw["combine"] = synth.COMBINE_SEPARATE
    if mode == "softplus":
        kw["dt_softplus"] = 1
    Dn = 256 if mode == "groups" else 96
    if mode == "groups":
        kw["n_groups"] = 2
    cfg = synth.mixer_cfg(3, 45, Dn, io="f32", **kw)
    run_case(gpu, oracle, cfg, 77, untied="untied" in mode, random_a=mode != "progression_a")


@pytest.mark.parametrize("seed", range(32))
def test_random_descriptor(gpu, oracle, seed):
    """Seeded random draws from the supported space: state count, conv width, length (around the chunks of 8 or 16 and
    the meeting point of the two walks), channel counts with ragged tiles and shadow waves, groups, modes, dtypes."""
    rng = np.random.default_rng(4100 + seed)
    N = int(rng.choice([4, 8, 16]))
    G = int(rng.choice([1, 1, 2]))
    Dn = int(rng.choice([128, 256, 384])) if G == 2 else int(rng.choice([1, 7, 64, 100, 130, 192, 200]))
    L = int(rng.choice([1, 2, 3, 5, 15, 17, 31, 33, 48, 65, 97]))
    cfg = synth.mixer_cfg(int(rng.integers(1, 4)), L, Dn, d_state=N, d_conv=int(rng.integers(1, 5)), n_groups=G,
                          io=str(rng.choice(["f32", "bf16"])), combine=int(rng.integers(0, 2)),
                          dt_softplus=int(rng.integers(0, 2)))
    run_case(gpu, oracle, cfg, 600 + seed, untied=bool(rng.integers(0, 2)), random_a=bool(rng.integers(0, 2)))


def test_gradient_call_replayed_from_a_hip_graph(gpu):
    """bimamba_bwd captured into a HIP graph (it enqueues kernels only): every replay, with eager work and synchronisation
    between replays and fresh contents in the static buffers, must equal the eager call on the same contents bit for bit
    (every sum has a fixed order)."""
    cfg = synth.mixer_cfg(3, 45, 200, io="bf16")
    Bt, L, Dn, N, K = 3, 45, 200, cfg["d_state"], cfg["d_conv"]
    pf, pb = params(cfg, 5)
    dpf, dpb = bd.to_device(pf), bd.to_device(pb)
    desc = bd.make_desc(cfg)
    static_in = bd.to_device(synth.make_inputs(cfg, 5), cfg)
    dout = torch.zeros(Bt, L, Dn, dtype=torch.bfloat16, device="cuda")
    io = torch.bfloat16
    gi = dict(dx=torch.empty(Bt, L, Dn, dtype=io, device="cuda"), dz=torch.empty(Bt, L, Dn, dtype=io, device="cuda"),
              ddt=torch.empty(Bt, L, Dn, dtype=io, device="cuda"), dB=torch.empty(Bt, L, 1, N, device="cuda"),
              dC=torch.empty(Bt, L, 1, N, device="cuda"))
    mk = lambda: dict(dconv_w=torch.empty(Dn, K, device="cuda"), dconv_b=torch.empty(Dn, device="cuda"),
                      dA=torch.empty(Dn, N, device="cuda"), dD=torch.empty(Dn, device="cuda"), ddt_bias=torch.empty(Dn, device="cuda"))
    qf, qb = mk(), mk()
    ws = torch.empty(bd.bimamba_bwd_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    args = (desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(static_in), None, bd.make_tensor(dout),
            bd.make_input_grads(gi), None, bd.make_param_grads(qf), bd.make_param_grads(qb), ws)

    def call():
        bd.bimamba_bwd(*args)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    outs = list(gi.values()) + list(qf.values()) + list(qb.values())
    for rep in range(3):
        fresh = bd.to_device(synth.make_inputs(cfg, 70 + rep), cfg)
        for k in static_in:
            static_in[k].copy_(fresh[k])
        dout.copy_(torch.randn(Bt, L, Dn, generator=torch.Generator().manual_seed(80 + rep)).to(io))
        call()
        torch.cuda.synchronize()
        want = [t.clone() for t in outs]
        for t in outs:
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for i, (got, ref) in enumerate(zip(outs, want)):
            assert torch.equal(got, ref), (rep, i)


@pytest.mark.parametrize("untied", [False, True])
def test_column_slices_with_their_own_token_strides(gpu, oracle, untied):
    """x, z, dt as column slices of one wide buffer per direction, dout a slice of another, dx, dz, ddt slices of a
    third: every tensor has its own row pitch, and the kernels step through each with its own stride.  Nothing outside
    the gradient views may be written."""
    cfg = synth.mixer_cfg(2, 37, 72, io="bf16", combine=synth.COMBINE_SEPARATE)
    Bt, L, Dn, N, K = 2, 37, 72, cfg["d_state"], cfg["d_conv"]
    io = torch.bfloat16
    pf, pb = params(cfg, 3)
    ins = [synth.make_inputs(cfg, 3)] + ([synth.make_inputs(cfg, 503)] if untied else [])
    g = torch.Generator().manual_seed(12)
    dout = rounded(torch.randn(Bt, L, 2 * Dn, generator=g), "bf16")

    def sliced(t, width, at):
        wide = torch.zeros(Bt, L, width, dtype=io, device="cuda")
        view = wide[..., at:at + t.shape[-1]]
        view.copy_(torch.as_tensor(t).to(io))
        return wide, view

    dev_in, grads, wides = [], [], []
    for inp in ins:
        d = bd.to_device(inp, cfg)
        d["x"] = sliced(inp["x"], 3 * Dn + 40, 8)[1]
        d["z"] = sliced(inp["z"], 2 * Dn + 24, 16)[1]
        d["dt"] = sliced(inp["dt"], Dn + 8, 0)[1]
        dev_in.append(d)
        wide = torch.zeros(Bt, L, 3 * Dn + 48, dtype=io, device="cuda")
        wides.append(wide)
        grads.append(dict(dx=wide[..., 8:8 + Dn], dz=wide[..., 16 + Dn:16 + 2 * Dn], ddt=wide[..., 40 + 2 * Dn:40 + 3 * Dn],
                          dB=torch.empty(Bt, L, 1, N, device="cuda"), dC=torch.empty(Bt, L, 1, N, device="cuda")))
    do = sliced(dout, 2 * Dn + 64, 32)[1]
    mk = lambda: dict(dconv_w=torch.empty(Dn, K, device="cuda"), dconv_b=torch.empty(Dn, device="cuda"),
                      dA=torch.empty(Dn, N, device="cuda"), dD=torch.empty(Dn, device="cuda"), ddt_bias=torch.empty(Dn, device="cuda"))
    qf, qb = mk(), mk()
    desc = bd.make_desc(cfg)
    dpf, dpb = bd.to_device(pf), bd.to_device(pb)
    ws = torch.empty(bd.bimamba_bwd_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    bd.bimamba_bwd(desc, bd.make_params(dpf), bd.make_params(dpb), bd.make_inputs(dev_in[0]),
                   bd.make_inputs(dev_in[1]) if untied else None, bd.make_tensor(do), bd.make_input_grads(grads[0]),
                   bd.make_input_grads(grads[1]) if untied else None, bd.make_param_grads(qf), bd.make_param_grads(qb), ws)
    torch.cuda.synchronize()
    host = lambda d: {k: v.float().cpu().numpy().astype(np.float64) for k, v in d.items()}
    got = (host(grads[0]), host(grads[1]) if untied else None, host(qf), host(qb))
    ref = oracle.bimamba_bwd(cfg, to_np(pf), to_np(pb), to_np(ins[0]), to_np(ins[1]) if untied else None, dout)
    compare(cfg, got, ref)
    for wide in wides:
        for lo, hi in ((0, 8), (8 + Dn, 16 + Dn), (16 + 2 * Dn, 40 + 2 * Dn), (40 + 3 * Dn, 48 + 3 * Dn)):
            assert float(wide[..., lo:hi].abs().max()) == 0.0


@pytest.mark.parametrize("untied", [False, True])
@pytest.mark.parametrize("L", [31, 63, 64, 65, 66, 67, 71, 127, 129, 130, 131, 193, 259, 517])
def test_lengths_around_the_time_segments(gpu, oracle, L, untied):
    """A small call is cut into time segments of whole chunks, 32 tokens or more: lengths at which the last segment is
    empty but for one to three tokens (the conv window and the dh window reach past it), odd chunk counts on either side
    of the meeting point, both decay forms, every conv width."""
    cfg = synth.mixer_cfg(2, L, 72, d_state=(16, 8, 4)[L % 3], d_conv=1 + L % 4, io="bf16", dt_softplus=L % 2)
    run_case(gpu, oracle, cfg, 40 + L, untied=untied, random_a=bool(L & 2))


@pytest.mark.parametrize("N", [4, 8, 16])
@pytest.mark.parametrize("L", [1, 5, 37, 70])
def test_more_waves_than_simds(gpu, oracle, N, L):
    """Batch 9 at d_inner 4096 is 1152 waves for 1024 SIMDs, in one or two time segments, and the plan that sizes their
    stored states; every channel compared."""
    run_case(gpu, oracle, synth.mixer_cfg(9, L, 4096, d_state=N, io="bf16" if L % 2 else "f32"), 900 + N + L)


def device_call(cfg, weights, acts, dout):
    """bimamba_bwd on tensors that are on the GPU already, both directions reading the same activations."""
    Bt, L, Dn, N, K = (cfg[k] for k in ("batch", "seqlen", "d_inner", "d_state", "d_conv"))
    io = bd.io_dtype(cfg)
    empty = lambda *s, dtype=torch.float32: torch.full(s, float("nan"), dtype=dtype, device="cuda")
    gi = dict(dx=empty(Bt, L, Dn, dtype=io), dz=empty(Bt, L, Dn, dtype=io), ddt=empty(Bt, L, Dn, dtype=io),
              dB=empty(Bt, L, 1, N), dC=empty(Bt, L, 1, N))
    qs = [dict(dconv_w=empty(Dn, K), dconv_b=empty(Dn), dA=empty(Dn, N), dD=empty(Dn), ddt_bias=empty(Dn)) for _ in range(2)]
    desc = bd.make_desc(cfg)
    dev = [bd.to_device(w) for w in weights]
    ws = torch.empty(bd.bimamba_bwd_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    bd.bimamba_bwd(desc, bd.make_params(dev[0]), bd.make_params(dev[1]), bd.make_inputs(acts), None, bd.make_tensor(dout),
                   bd.make_input_grads(gi), None, bd.make_param_grads(qs[0]), bd.make_param_grads(qs[1]), ws)
    torch.cuda.synchronize()
    return gi, qs


@pytest.mark.parametrize("N", [4, 8, 16])
def test_a_channel_does_not_feel_its_neighbours_decay_rates(gpu, N):
    """A channel's gradients depend on its own A row alone: with the rows of the other channels of its wave arithmetic in n
    (as at initialisation) or not (as training leaves them), its fp32 gradients have the same bits, i.e. there is no second,
    less exact form of the decay factors for waves whose rows are all arithmetic."""
    cfg = synth.mixer_cfg(2, 150, 128, d_state=N, io="bf16", dt_softplus=1)
    pf, pb = params(cfg, 5, random_a=False)
    acts = bd.to_device(synth.make_inputs(cfg, 5), cfg)
    dout = torch.randn(2, 150, 128, generator=torch.Generator().manual_seed(6)).to("cuda", torch.bfloat16)
    before = device_call(cfg, (pf, pb), acts, dout)
    touched = [5, 70]                    # one channel of each wave
    for p in (pf, pb):
        p["A"][touched] = p["A"][touched] * torch.linspace(0.8, 1.3, N)
    after = device_call(cfg, (pf, pb), acts, dout)
    keep = [c for c in range(128) if c not in touched]
    for k in ("dx", "dz", "ddt"):
        assert torch.equal(before[0][k][..., keep], after[0][k][..., keep]), k
    for s in range(2):
        for k in before[1][s]:
            assert torch.equal(before[1][s][k][keep], after[1][s][k][keep]), (s, k)
        assert not torch.equal(before[1][s]["dA"][touched], after[1][s]["dA"][touched])


@pytest.mark.parametrize("io,random_a", [("bf16", False), ("bf16", True), ("f32", True)])
def test_long_time_segments(gpu, oracle, io, random_a):
    """8 x 8192 tokens of 4096 channels: segments of 1024 tokens, whose dh sums decay over far larger sums of Delta than
    those of small calls.  dout is zero but for eight channels, so that the sums over channels are theirs alone and the
    oracle needs only them."""
    Bt, L, Dn = 8, 8192, 4096
    cfg = synth.mixer_cfg(Bt, L, Dn, io=io)
    weights = params(cfg, 15, random_a=random_a)
    sel = [0, 63, 64, 130, 1000, 2047, 4000, 4095]
    g = torch.Generator(device="cuda").manual_seed(16)
    dtype = bd.io_dtype(cfg)
    normal = lambda n: torch.randn(Bt, L, n, device="cuda", generator=g).to(dtype)
    acts = dict(x=normal(Dn), z=normal(Dn), B=normal(16), C=normal(16))
    acts["dt"] = torch.nn.functional.softplus(0.5 * torch.randn(Bt, L, Dn, device="cuda", generator=g) +
                                              synth.dt_shift(cfg, 15).cuda()).to(dtype)
    dout = torch.zeros(Bt, L, Dn, dtype=dtype, device="cuda")
    dout[..., sel] = normal(len(sel))
    gi, qs = device_call(cfg, weights, acts, dout)
    host = lambda t: t.float().cpu().numpy().astype(np.float64)
    got_in = {k: host(v[..., sel]) if k in ("dx", "dz", "ddt") else host(v) for k, v in gi.items()}
    got_par = [{k: host(v[sel]) for k, v in q.items()} for q in qs]
    for k in ("dx", "dz", "ddt"):        # the other channels' gradients are zero
        others = gi[k].clone()
        others[..., sel] = 0
        assert not bool(others.any()), k
    inp = {k: host(v[..., sel]) if k in ("x", "z", "dt") else host(v).reshape(Bt, L, 1, 16) for k, v in acts.items()}
    small = synth.mixer_cfg(Bt, L, len(sel), io=io)
    cut = [{k: None if v is None else to_np({k: v})[k][sel] for k, v in w.items()} for w in weights]
    ref = oracle.bimamba_bwd(small, cut[0], cut[1], inp, None, host(dout[..., sel]))
    compare(small, (got_in, None, *got_par), ref)


def test_empty_call_zeroes_the_parameter_gradients(gpu, oracle):
    cfg = synth.mixer_cfg(0, 16, 64, io="f32")
    pf, pb = params(cfg, 1)
    got = gpu.gpu_bwd(cfg, pf, pb, synth.make_inputs(cfg, 1), None, np.zeros((0, 16, 64), dtype=np.float32))
    assert got[0]["dx"].shape == (0, 16, 64)
    for q in got[2:]:
        assert all(not np.any(v) for v in q.values())


def test_unsupported_layouts_are_refused_on_the_host(gpu):
    for cfg in (synth.m2_cfg(1, 64, 128, headdim=64, d_state=64), synth.mixer_cfg(1, 8, 64, d_state=32)):
        assert bd.bimamba_bwd_workspace_bytes(bd.make_desc(cfg)) == 0


def test_headline_width_sampled(gpu, oracle):
    """d_inner 4096, bf16, a few hundred tokens: the x / z / Delta and per-channel parameter gradients on sampled
    channels (B and C gradients are sums over all channels and are covered by the small cases)."""
    cfg = synth.mixer_cfg(2, 300, 4096)
    pf, pb = params(cfg, 5, random_a=False)
    inp = synth.make_inputs(cfg, 5)
    g = torch.Generator().manual_seed(3)
    dout = rounded(torch.randn(2, 300, 4096, generator=g), "bf16")
    sel = list(range(3, 4096, 511))
    got = gpu.gpu_bwd(cfg, pf, pb, inp, None, dout)
    ref = oracle.bimamba_bwd(cfg, to_np(pf), to_np(pb), to_np(inp), None, dout[..., sel], sel=sel)
    compare(cfg, got, ref, sel=sel)


def test_sum_over_a_segment_rounds_no_more_than_term_by_term(gpu, oracle):
    """What a segment's tokens add to the dh of the tokens before it.  With an output gradient in the last 29 of 64 tokens only (a segment of
    32 whose sum starts three tokens in) dB of the four tokens before the segment is that sum, a few decays and a product, of one
    channel and here of gates and conv outputs that no rounding touches (SiLU of 20 and more).  It is no further from 64 bits than the
    same in fp32 with the sum formed term by term and every exponential correctly rounded."""
    batch, L, N, seg = 1024, 64, 16, 35
    cfg = synth.mixer_cfg(batch, L, 1, d_state=N, io="f32", d_conv=1)
    pf, pb = synth.make_params(cfg, 5, 0), synth.make_params(cfg, 5, 1)
    inp, inp_b = synth.make_inputs(cfg, 5), synth.make_inputs(cfg, 6)
    for p in (pf, pb):
        p["conv_w"].fill_(1.0)
        p["conv_b"].zero_()
    g = torch.Generator().manual_seed(5)
    for i in (inp, inp_b):
        for k in ("x", "z"):
            i[k].uniform_(20.0, 40.0, generator=g)
    # (one channel: the batch elements bring the spread of rates that channels have)
    inp["dt"] *= torch.exp(2.0 * torch.rand(batch, 1, 1, generator=g) - 1.0)
    dout = np.zeros((batch, L, 1), dtype=np.float32)
    dout[:, seg:] = np.random.default_rng(5).standard_normal((batch, L - seg, 1))
    got = gpu.gpu_bwd(cfg, pf, pb, inp, inp_b, dout)[0]["dB"][:, 28:32, 0]
    ref = oracle.bimamba_bwd(cfg, to_np(pf), to_np(pb), to_np(inp), to_np(inp_b), dout)[0]["dB"][:, 28:32, 0]
    x, z, dt, C = (inp[k].numpy().reshape(batch, L, -1) for k in ("x", "z", "dt", "C"))
    a2 = (pf["A"].numpy()[0] * np.float32(np.log2(np.e))).astype(np.float32)
    decay = lambda w: np.exp2((w * a2).astype(np.float64)).astype(np.float32)
    dh, w = np.zeros((batch, N), np.float32), np.zeros((batch, 1), np.float32)
    for t in range(seg, L):
        w = w + dt[:, t]
        dh = ((dout[:, t] * z[:, t] * decay(w)).astype(np.float64) * C[:, t] + dh).astype(np.float32)
    plain = np.empty_like(got)
    for t in range(seg - 1, 27, -1):
        if t < 32:
            plain[:, t - 28] = dh * (dt[:, t] * x[:, t])
        dh = dh * decay(dt[:, t])
    assert rel_all(got, ref) < rel_all(plain, ref), (rel_all(got, ref), rel_all(plain, ref))
