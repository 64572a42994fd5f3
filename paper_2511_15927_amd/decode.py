"""Block-diffusion decode loop around bimamba_block_fwd (paper Sec. 4.3, block-cache decoding).

A block of G tokens is denoised in n_steps = G / p steps (Sec. 4.3 throughput set-up: p tokens per step); at every
step all n_layers mixer layers re-scan the block from their cached forward state, the reverse scan staying inside the
block; the last step commits each layer's state and conv tail, which the next block starts from.  This module only
sequences library calls and owns the buffers: every scan runs in the HIP library.

Layer chaining of this benchmark stack (no projections between the mixers are part of the path): layer l's output is
layer l+1's x; z, dt, B, C of a step are shared by the layers; parameters are per layer and per direction.

The n_steps x n_layers calls of a block are captured ONCE into a HIP graph (torch.cuda.CUDAGraph: stream capture of
the library's launches, which contain no memset nodes) and replayed per block; the caller refreshes the static step
inputs between replays.  Nothing on this path mixes channels, so with few enough chains the whole block is one launch in which a
workgroup takes a few channels through every layer of every step (bimamba_block_stack; at batch 1, 24 layers x 8 steps of 32
tokens 1.44 -> 0.26 ms with the refresh of the step inputs).  Otherwise the state of all layers (n_layers x batch x d_inner x d_state fp32, 100 MB at batch 16)
lives in HBM/L2 between calls and a call reads it once (4 MB per layer call against 8 MB of activations).
"""
import torch

from . import binding as bd
from . import synth


class BlockDecodeLoop:
    def __init__(self, cfg, layer_params, n_steps, keep_layer_outputs=False, static_scratch=False, device="cuda"):
        """cfg: block config (seqlen = G); layer_params: list of (params_f, params_b) dicts of CPU float32 tensors.
        static_scratch: the calls take the library's fixed scratch, not a workspace (a block in one launch needs neither)."""
        self.cfg, self.n_layers, self.n_steps = dict(cfg), len(layer_params), int(n_steps)
        self.desc = bd.make_desc(cfg)
        Bt, G, Dn, N, K = cfg["batch"], cfg["seqlen"], cfg["d_inner"], cfg["d_state"], cfg["d_conv"]
        io = bd.io_dtype(cfg)
        tail_ch = synth.conv_channels(cfg)
        self._dev_params = [(bd.to_device(pf, device=device), bd.to_device(pb, device=device)) for pf, pb in layer_params]
        self._params = [(bd.make_params(f), bd.make_params(b)) for f, b in self._dev_params]
        self.h = [torch.zeros(Bt, Dn, N, dtype=torch.float32, device=device) for _ in range(self.n_layers)]
        self.tail = [torch.zeros(Bt, max(K - 1, 1), tail_ch, dtype=io, device=device)[:, :K - 1].contiguous()
                     for _ in range(self.n_layers)]
        H, GN = cfg["n_heads"], cfg["n_groups"] * N
        # static inputs of each step (the caller writes the block's current tokens here before a block runs)
        # A step's tensors lie one behind the other.
        widths = dict(x=Dn, z=Dn, dt=H, B=GN, C=GN)
        self._step_flat = [torch.zeros(Bt * G * sum(widths.values()), dtype=io, device=device) for _ in range(self.n_steps)]
        self.step_inputs = [{k: t.view(Bt, G, n) for (k, n), t in zip(widths.items(), flat.split([Bt * G * n for n in widths.values()]))}
                            for flat in self._step_flat]
        self._step_views = [dict(views) for views in self.step_inputs]
        self._row_strides = {k: (G * n, n) for k, n in widths.items()}
        self._step_places = [bd.make_inputs(views) for views in self.step_inputs]
        self._step_ptrs = [{k: t.data_ptr() for k, t in views.items()} for views in self.step_inputs]
        self._device = self._step_flat[0].get_device() if self.n_steps else -1   # (-1: host memory)
        self._copies_at_once = self._device >= 0
        width = Dn * (2 if cfg["combine"] == bd.COMBINE_SEPARATE else 1)
        assert width == Dn, "layers chain out -> x, which needs the additive combine"
        n_act = self.n_steps * self.n_layers if keep_layer_outputs else 2
        self._act = [torch.zeros(Bt, G, Dn, dtype=io, device=device) for _ in range(n_act)]
        self.keep = keep_layer_outputs
        self.out = [torch.zeros(Bt, G, Dn, dtype=io, device=device) for _ in range(self.n_steps)]   # last layer, per step
        self.static_scratch = static_scratch
        self.ws = None if static_scratch else bd.alloc_workspace(self.desc, 1, device=device)
        self._graph = None
        # few enough chains: the whole block is one launch (bimamba_block_stack), whose table of pointers sits on the device
        self._one_launch = self.n_layers > 0 and self.n_steps > 0 and bd.bimamba_block_stack_form(self.desc) == 1
        # (uploaded here: under a caller's own capture, which the first run may be, it could not be)
        self._table, self._table_dev, self._captured = None, None, []
        if self._one_launch:
            self._upload(self._stack_table())

    def layer_output(self, step, layer):
        assert self.keep
        return self.out[step] if layer == self.n_layers - 1 else self._act[step * self.n_layers + layer]

    def set_step_inputs(self, step, inputs):
        """inputs: dict of tensors x, z [Bt,G,Dn]; dt [Bt,G,H]; B, C [Bt,G,G*N] or [Bt,G,groups,N] (any device)."""
        if self._copies_at_once and self._device != torch.cuda.current_device():
            with torch.cuda.device(self._device):
                return self.set_step_inputs(step, inputs)
        dsts = self.step_inputs[step]
        if not self._copies_at_once or not self._copy_at_once(step, dsts, inputs):
            for k, dst in dsts.items():
                dst.copy_(inputs[k].reshape(dst.shape))

    def _copy_at_once(self, step, dsts, inputs):
        """A step's tensors in one launch, where they are of the buffer's kind and no part of it and it stands where it was made; one that
        does not lie in rows of whole channels is copied into such rows before.  False: nothing was written.  (24 layers x 8 steps of 32
        tokens at batch 1: 57 us of host time a step with one concatenation, 12 so.)"""
        flat, views, places, words, held = self._step_flat[step], self._step_views[step], self._step_ptrs[step], [], []
        if flat.is_inference() and not torch.is_inference_mode_enabled():
            return False   # (a write that torch refuses)

        def in_rows(t, dst):
            return (t.dim() == 3 and t.shape == dst.shape and t.stride(2) == 1 and t.stride(1) >= t.shape[2] and
                    (t.shape[0] == 1 or t.stride(0) >= (t.shape[1] - 1) * t.stride(1) + t.shape[2]))

        for k, dst in dsts.items():
            t = inputs[k]
            if (dst is not views[k] or dst.data_ptr() != places[k] or type(t) not in (torch.Tensor, torch.nn.Parameter) or t.get_device() != self._device or
                    t.dtype is not flat.dtype or t.numel() != dst.numel() or t.requires_grad or t.is_neg()):
                return False
            if t.is_contiguous():
                words += (t.data_ptr(), *self._row_strides[k])
                continue
            if not in_rows(t, dst):
                if t.untyped_storage().data_ptr() == flat.untyped_storage().data_ptr():
                    return False   # (to be read after the tensors before it are written)
                t = t.reshape(dst.shape)
                t = t if in_rows(t, dst) else t.contiguous()
                held.append(t)
            words += (t.data_ptr(), t.stride(0), t.stride(1))
        if bd.bimamba_copy_inputs(self.desc, bd.input_words(words), self._step_places[step], check=False) != 0:
            return False   # (a part of the buffer among them)
        torch.autograd.graph.increment_version(flat)
        return True

    def _call(self, layer, step, x, out, commit, stream):
        pf, pb = self._params[layer]
        si = self.step_inputs[step]
        ins = bd.make_inputs(dict(x=x, z=si["z"], dt=si["dt"], B=si["B"], C=si["C"]))
        h, tail = self.h[layer], self.tail[layer]
        has_tail = tail.shape[1] > 0
        a = (self.desc, pf, pb, ins, None, h, tail if has_tail else None, h if commit else None,
             tail if (commit and has_tail) else None, bd.make_tensor(out))
        if self.static_scratch:
            bd.bimamba_block_fwd_static(*a, stream=stream)
        else:
            bd.bimamba_block_fwd(*a, self.ws, stream=stream)

    def _stack_table(self):
        """The pointers bimamba_block_stack works from."""
        has_tail = self.tail[0].shape[1] > 0
        layers = [bd.StackLayer(pf, pb, h.data_ptr(), t.data_ptr() if has_tail else None)
                  for (pf, pb), h, t in zip(self._params, self.h, self.tail)]
        steps = [bd.make_inputs(s) for s in self.step_inputs]
        outs = [self.out[s] if l == self.n_layers - 1 else self._act[s * self.n_layers + l] if self.keep else None
                for s in range(self.n_steps) for l in range(self.n_layers)]
        return bd.make_stack_table(layers, steps, outs)

    def _upload(self, table):
        dev = torch.frombuffer(bytearray(table), dtype=torch.uint8).to(self.out[0].device)
        if self._table_dev is not None:
            torch.cuda.synchronize()   # (launches that read the one before have run)
        self._table, self._table_dev = table, dev

    def _run_stack(self, stream):
        """The whole block in one launch.  False: the tensors have changed since the table was uploaded, and a stream that is being
        captured cannot upload it anew."""
        table = self._stack_table()
        with torch.cuda.stream(stream):
            capturing = torch.cuda.is_current_stream_capturing()
        if table != self._table:
            if capturing:
                return False
            self._upload(table)
        if capturing and not any(t is self._table_dev for t in self._captured):
            self._captured.append(self._table_dev)   # the captured launch reads it at every replay
        bd.bimamba_block_stack(self.desc, self.n_layers, self.n_steps, self._table, self._table_dev, stream=stream)
        return True

    def run_block_eager(self, stream=None):
        """All steps of one block, call by call (in one launch where the library can); the last step commits every layer's
        state and conv tail in place."""
        if self._one_launch and self._run_stack(stream):
            return
        for step in range(self.n_steps):
            commit = step == self.n_steps - 1
            x = self.step_inputs[step]["x"]
            for layer in range(self.n_layers):
                last = layer == self.n_layers - 1
                out = self.out[step] if last else (self._act[step * self.n_layers + layer] if self.keep else self._act[layer & 1])
                self._call(layer, step, x, out, commit, stream)
                x = out

    def capture(self):
        """Capture one block's calls into a graph (after one eager pass on a side stream, so that no kernel variant
        is launched for the first time under capture and the cache is left as it was)."""
        saved = [(h.clone(), t.clone()) for h, t in zip(self.h, self.tail)]
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            self.run_block_eager()
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        for (h0, t0), h, t in zip(saved, self.h, self.tail):
            h.copy_(h0)
            t.copy_(t0)
        self._graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self._graph):
            self.run_block_eager()
        # the capture itself does not run the kernels: the cache is untouched
        return self

    def run_block(self):
        """Replay the captured block (capture() first)."""
        self._graph.replay()

    def prefill(self, make_layer_inputs, prefix_len):
        """Scan a clean prefix once through every layer, committing each layer's state and conv tail.
        make_layer_inputs: dict of device tensors for the prefix (x of layer 0, z, dt, B, C)."""
        cfg_p = dict(self.cfg, seqlen=prefix_len)
        desc = bd.make_desc(cfg_p)
        ws = bd.alloc_workspace(desc, 1)
        x = make_layer_inputs["x"]
        for layer in range(self.n_layers):
            pf, pb = self._params[layer]
            out = torch.empty_like(make_layer_inputs["x"])
            ins = bd.make_inputs(dict(make_layer_inputs, x=x))
            tail = self.tail[layer]
            bd.bimamba_block_fwd(desc, pf, pb, ins, None, None, None, self.h[layer], tail if tail.shape[1] > 0 else None,
                                 bd.make_tensor(out), ws)
            x = out
        torch.cuda.synchronize()
        return x
