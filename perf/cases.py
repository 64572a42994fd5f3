"""What this framework is timed on: calls of its public entry points at the sizes its users run.

Four kinds of call, each in the parameterisations that have it:
  fwd     bimamba_fwd, a full-sequence denoising step of one mixer layer (and the forward half of a training step);
  block   bimamba_block_fwd, one layer of block diffusion: a denoising step of a short block from the cached state, or the
          scan of a clean prefix that fills the cache;
  decode  BlockDecodeLoop.run_block, a block of tokens through every denoising step of a stack of layers;
  bwd     bimamba_bwd, the gradients of a training step.
"selective" is the selective-scan layout (Delta, A and D per channel), "mamba2" the paper's layout (one Delta, A and D
per head, conv on B and C too).  Fields of a case: `untied`: each direction has activations of its own (the paper's
setting; the two outputs are then kept apart for their two output projections); `packed`: the activations are column
slices of the projection outputs that hold them, as a model hands them over; `trained_A`: decay rates with no structure
across states, as training leaves them, against the initial -(1..N); `softplus`: Delta comes raw, with its bias;
`commit`: the call also writes the state and conv tail that the next block starts from.
"""
import math

import torch

from paper_2511_15927_amd import binding as bd
from paper_2511_15927_amd import shapes, synth
from paper_2511_15927_amd.decode import BlockDecodeLoop

_BASE = dict(kind="fwd", form="selective", batch=1, seqlen=1024, d_inner=4096, d_state=16, headdim=1, io="bf16", softplus=0,
             untied=0, packed=0, trained_A=0, commit=0, layers=1, steps=1)


def _case(name=None, **kw):
    c = dict(_BASE, **kw)
    if c["form"] == "mamba2":
        c["softplus"] = 1
    return c if name is None else dict(name=name, **c)


def listed():
    return [
        # the smallest call: a small fp32 mixer as one trains and checks a toy model with (configuration 0)
        _case("tiny_fp32", seqlen=256, d_inner=512, io="f32"),
        # one layer of a 1.3B-scale model in a denoising step, trained weights, x | z and B | C as their projections leave them
        _case("layer_b8_trained", batch=8, seqlen=2048, trained_A=1, packed=1),
        # the benchmark's headline call
        _case("headline", batch=8, seqlen=8192),
        # a single long sequence, the regime in which the paper reports its largest speed-ups (configuration 2)
        _case("long_b1", seqlen=32768),
        # sizes nobody tuned for: a ragged width and length, both directions with activations of their own, raw Delta
        _case("ragged_untied", batch=3, seqlen=1237, d_inner=1480, softplus=1, untied=1, packed=1),
        # the paper's 1.3B layer at the batch and length of interactive use, as its in_proj hands the activations over
        _case("m2_paper_b1", form="mamba2", seqlen=1024, d_inner=3840, d_state=128, headdim=32, untied=1, packed=1),
        # the headline call in the paper's parameterisation
        _case("m2_headline", form="mamba2", batch=8, seqlen=8192, d_state=128, headdim=64),
        # block diffusion: the last denoising step of a 32-token block, which commits the cache
        _case("block_step", kind="block", batch=16, seqlen=32, commit=1),
        # block diffusion in the paper's parameterisation: a step that leaves the cache as it is
        _case("m2_block_step", kind="block", form="mamba2", batch=16, seqlen=32, d_state=128, headdim=64),
        # a user generating one sequence: 32 tokens through 8 denoising steps of 24 layers, one graph replay
        _case("decode_b1", kind="decode", batch=1, seqlen=32, layers=24, steps=8),
        # training: gradients of the headline call, the largest amount of work here
        _case("bwd_headline", kind="bwd", batch=8, seqlen=8192),
        # training a small model on ragged sequences, each direction with activations of its own
        _case("bwd_small_untied", kind="bwd", batch=4, seqlen=771, d_inner=1536, softplus=1, untied=1, trained_A=1),
    ]


_MOST_STATE_STEPS = 8 * 8192 * 4096 * 16   # batch * tokens * channels * states of the headline call


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fwd", "fwd", "fwd", "block", "block", "decode", "bwd", "bwd"])
    form = "selective" if kind == "bwd" else rng.choice(["selective", "mamba2"])
    c = dict(kind=kind, form=form, untied=rng.randint(0, 1), packed=rng.randint(0, 1), trained_A=rng.randint(0, 1),
             softplus=rng.randint(0, 1))
    if form == "selective":
        c["d_inner"] = _log_int(rng, 512, 4096) // 8 * 8
        c["d_state"] = rng.choice([16, 16, 16, 8])
        c["io"] = rng.choice(["bf16", "bf16", "bf16", "f32"])
        states = c["d_state"]
    else:
        c["headdim"] = rng.choice([32, 64])
        c["d_inner"] = max(1, _log_int(rng, 512, 4096) // c["headdim"]) * c["headdim"]
        c["d_state"] = rng.choice([64, 128, 128])
        states = 16   # the matrix-core path: its cost follows the tokens and channels
    if kind == "decode":
        c.update(batch=_log_int(rng, 1, 16), seqlen=rng.choice([16, 32, 32, 64]), layers=rng.randint(4, 24), steps=rng.randint(2, 8),
                 io="bf16", untied=0, packed=0)
        return _case(**c)
    if kind == "block":
        c["commit"] = rng.randint(0, 1)
        c["seqlen"] = _log_int(rng, 16, 128) if rng.random() < 0.7 else _log_int(rng, 128, 4096)
        c["batch"] = _log_int(rng, 1, 32)
    elif kind == "bwd":
        c["seqlen"] = _log_int(rng, 128, 8192)
        c["batch"] = _log_int(rng, 1, 32)
    else:
        c["seqlen"] = _log_int(rng, 64, 32768)
        c["batch"] = _log_int(rng, 1, 64)
    room = _MOST_STATE_STEPS // (c["batch"] * c["d_inner"] * states * (2 if c["untied"] else 1))
    c["seqlen"] = max(16, min(c["seqlen"], room))
    return _case(**c)


def _cfg(c):
    combine = synth.COMBINE_SEPARATE if c["untied"] else synth.COMBINE_ADD
    if c["form"] == "mamba2":
        return synth.m2_cfg(c["batch"], c["seqlen"], c["d_inner"], headdim=c["headdim"], d_state=c["d_state"], io=c["io"],
                            combine=combine)
    return synth.mixer_cfg(c["batch"], c["seqlen"], c["d_inner"], d_state=c["d_state"], io=c["io"], combine=combine,
                           dt_softplus=c["softplus"])


def _params(c, cfg, seed, direction):
    p = synth.make_params(cfg, seed, direction)
    if c["trained_A"]:
        p["A"] = synth.random_A(cfg, 2 * seed + direction)
    return p


def _activations(c, cfg, gen, seed):
    """x, z, dt, B, C of one direction on the GPU, with the distributions of synth.make_inputs; packed: x and z (and, in
    the paper's layout, B, C and dt too) are column slices of one projection output."""
    io = bd.io_dtype(cfg)
    Bt, L, Dn, H, GN = cfg["batch"], cfg["seqlen"], cfg["d_inner"], cfg["n_heads"], cfg["n_groups"] * cfg["d_state"]

    def normal(n, scale=1.0):
        return (scale * torch.randn(Bt, L, n, device="cuda", generator=gen)).to(io)

    if c["packed"] and c["form"] == "mamba2":   # in_proj of the Mamba-2 layer: z | x | B | C | dt
        proj = normal(2 * Dn + 2 * GN + H)
        z, x, B, C, dt = proj.split([Dn, Dn, GN, GN, H], dim=2)
        dt.mul_(0.5)
        return dict(x=x, z=z, dt=dt, B=B, C=C)
    if c["packed"]:   # in_proj: x | z; x_proj: low-rank dt | B | C, the former on to dt_proj
        rank = (Dn + 31) // 32
        xz, low = normal(2 * Dn), normal(rank + 2 * GN)
        x, z = xz.split([Dn, Dn], dim=2)
        B, C = low[..., rank:rank + GN], low[..., rank + GN:]
    else:
        x, z, B, C = normal(Dn), normal(Dn), normal(GN), normal(GN)
    dt = 0.5 * torch.randn(Bt, L, H, device="cuda", generator=gen)
    if not cfg["dt_softplus"]:
        dt = torch.nn.functional.softplus(dt + synth.dt_shift(cfg, seed).cuda())
    return dict(x=x, z=z, dt=dt.to(io), B=B, C=C)


def _empty_grads(cfg):
    io = bd.io_dtype(cfg)
    Bt, L, Dn, G, N, K = (cfg[k] for k in ("batch", "seqlen", "d_inner", "n_groups", "d_state", "d_conv"))
    act = dict(dx=torch.empty(Bt, L, Dn, dtype=io, device="cuda"), dz=torch.empty(Bt, L, Dn, dtype=io, device="cuda"),
               ddt=torch.empty(Bt, L, Dn, dtype=io, device="cuda"), dB=torch.empty(Bt, L, G, N, device="cuda"),
               dC=torch.empty(Bt, L, G, N, device="cuda"))
    par = [dict(dconv_w=torch.empty(Dn, K, device="cuda"), dconv_b=torch.empty(Dn, device="cuda"), dA=torch.empty(Dn, N, device="cuda"),
                dD=torch.empty(Dn, device="cuda"), ddt_bias=torch.empty(Dn, device="cuda")) for _ in range(2)]
    return act, par


def prepare(case, seed):
    c = dict(_BASE, **case)
    cfg = _cfg(c)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    s = dict(kind=c["kind"])
    if c["kind"] == "decode":
        layers = [(_params(c, cfg, seed * 1000 + l, 0), _params(c, cfg, seed * 1000 + l, 1)) for l in range(c["layers"])]
        loop = BlockDecodeLoop(cfg, layers, c["steps"])
        for h in loop.h:
            h.copy_(0.2 * torch.randn(h.shape, device="cuda", generator=gen))
        for t in loop.tail:
            t.copy_(torch.randn(t.shape, device="cuda", generator=gen))
        s["tokens"] = [_activations(c, cfg, gen, seed) for _ in range(c["steps"])]
        s["loop"] = loop.capture()
        return s
    s["desc"] = bd.make_desc(cfg)
    s["weights"] = [bd.to_device(_params(c, cfg, seed, d)) for d in (0, 1)]
    s["pf"], s["pb"] = bd.make_params(s["weights"][0]), bd.make_params(s["weights"][1])
    s["in_f"] = _activations(c, cfg, gen, seed)
    s["in_b"] = _activations(c, cfg, gen, seed) if c["untied"] else None
    Bt, Dn, N, K = cfg["batch"], cfg["d_inner"], cfg["d_state"], cfg["d_conv"]
    if c["kind"] == "bwd":
        s["dout"] = torch.randn(bd.alloc_out(cfg).shape, device="cuda", generator=gen).to(bd.io_dtype(cfg))
        s["grads_f"], s["param_grads"] = _empty_grads(cfg)
        s["grads_b"] = _empty_grads(cfg)[0] if c["untied"] else None
        s["ws"] = torch.empty(bd.bimamba_bwd_workspace_bytes(s["desc"]), dtype=torch.uint8, device="cuda")
        return s
    s["out"] = bd.alloc_out(cfg)
    s["ws"] = bd.alloc_workspace(s["desc"], 1 if c["kind"] == "block" else 0)
    if c["kind"] == "block":
        channels = synth.conv_channels(cfg)
        s["h"] = 0.2 * torch.randn(Bt, Dn, N, device="cuda", generator=gen)
        s["tail"] = torch.randn(Bt, K - 1, channels, device="cuda", generator=gen).to(bd.io_dtype(cfg))
        s["h_out"] = torch.empty_like(s["h"]) if c["commit"] else None
        s["tail_out"] = torch.empty_like(s["tail"]) if c["commit"] else None
    return s


def run(state):
    s = state
    if s["kind"] == "decode":
        loop = s["loop"]
        for k, tokens in enumerate(s["tokens"]):
            loop.set_step_inputs(k, tokens)
        loop.run_block()
        return dict(out=loop.out, h=loop.h, tail=loop.tail)
    in_f = bd.make_inputs(s["in_f"])
    in_b = None if s["in_b"] is None else bd.make_inputs(s["in_b"])
    if s["kind"] == "bwd":
        bd.bimamba_bwd(s["desc"], s["pf"], s["pb"], in_f, in_b, bd.make_tensor(s["dout"]), bd.make_input_grads(s["grads_f"]),
                       None if in_b is None else bd.make_input_grads(s["grads_b"]), bd.make_param_grads(s["param_grads"][0]),
                       bd.make_param_grads(s["param_grads"][1]), s["ws"])
        return dict(f=s["grads_f"], b=s["grads_b"], params=s["param_grads"])
    if s["kind"] == "block":
        bd.bimamba_block_fwd(s["desc"], s["pf"], s["pb"], in_f, in_b, s["h"], s["tail"], s["h_out"], s["tail_out"],
                             bd.make_tensor(s["out"]), s["ws"])
        return dict(out=s["out"], h=s["h_out"], tail=s["tail_out"])
    bd.bimamba_fwd(s["desc"], s["pf"], s["pb"], in_f, in_b, bd.make_tensor(s["out"]), s["ws"])
    return s["out"]


def work(case):
    c = dict(_BASE, **case)
    cfg = _cfg(c)
    calls = c["layers"] * c["steps"]
    if c["kind"] == "bwd":
        return dict(bytes=shapes.algorithmic_bytes_bwd(cfg, shared_inputs=not c["untied"]), flops=shapes.algorithmic_flops_bwd(cfg))
    flops = shapes.ssd_matrix_flops(cfg) if c["form"] == "mamba2" else shapes.algorithmic_flops(cfg)
    nbytes = shapes.algorithmic_bytes(cfg, shared_inputs=not c["untied"])
    state = 4 * cfg["batch"] * cfg["d_inner"] * cfg["d_state"]
    if c["kind"] == "block":
        nbytes += state * (1 + c["commit"])
    elif c["kind"] == "decode":   # every layer's state is read in every step and written in the last one
        nbytes += state + state // c["steps"]
    return dict(bytes=calls * nbytes, flops=calls * flops)


def tolerance(case):
    c = dict(_BASE, **case)
    if c["io"] == "f32" and c["form"] == "selective":
        return {"rel": 1e-5}
    return {"rel": 1e-2}   # bf16 activations, and bf16 matrix operands in the paper's layout
