"""Host-side step driver: walks a layer manifest and issues the C-ABI calls of one DP-SGD step
(Algorithm 1: per-example clip, sum over the micro-batch, accumulate over micro-batches, then noise
and the Adam update with decoupled weight decay).  Host logic only: every computation is a library call."""
from __future__ import annotations

from . import binding as B_


def _elements(shape):
    n = 1
    for s in shape:
        n *= s
    return n


class StepRunner:
    """Owns the flat fp32 state (theta, m, v, clip-weighted sum S) of a manifest and the per-example
    squared-norm buffer.  Tensors of the flat space follow the manifest order (LayerSpec.tensors())."""

    def __init__(self, ctx, manifest, max_batch, device="cuda:0"):
        import torch

        self.ctx = ctx
        self.manifest = manifest
        self.offsets = []  # per layer: list of (offset, shape)
        off = 0
        for spec in manifest:
            cur = []
            for _, shp in spec.tensors():
                off = (off + 3) // 4 * 4  # keep every tensor 16-byte aligned inside the flat buffers
                cur.append((off, shp))
                off += _elements(shp)
            self.offsets.append(cur)
        self.P = off
        # byte offsets of the tensors inside a flat buffer: what the batched calls need of a layer's sums
        self._at = [[4 * o for o, _ in cur] for cur in self.offsets]
        self._spans = [[(4 * o, _elements(shp)) for o, shp in cur] for cur in self.offsets]  # ... and their elements
        self.S = torch.zeros(self.P, dtype=torch.float32, device=device)
        self.theta = torch.zeros(self.P, dtype=torch.float32, device=device)
        self.m = torch.zeros(self.P, dtype=torch.float32, device=device)
        self.v = torch.zeros(self.P, dtype=torch.float32, device=device)
        self.sqnorms = torch.zeros(max_batch, dtype=torch.float32, device=device)
        # per-example LayerNorm gradients kept from pass 1 for pass 2 (2 d floats per example and layer)
        self.max_batch = max_batch
        self.device = device
        self.ln_keep = {}
        self._kept_for = None

    def view(self, buf, layer, k):
        off, shp = self.offsets[layer][k]
        return buf[off:off + _elements(shp)].view(*shp)

    def _keep_buffer(self, k, d):
        """[max_batch, 2, d] floats for layer k of the manifest, allocated on first use."""
        import torch

        buf = self.ln_keep.get(k)
        if buf is None or buf.numel() < self.max_batch * 2 * d:
            buf = torch.empty(self.max_batch * 2 * d, dtype=torch.float32, device=self.device)
            self.ln_keep[k] = buf
        return buf

    @staticmethod
    def _ln_token(layers, nB):
        """Identifies the micro-batch whose LayerNorm gradients the keep buffers hold: batch size and input buffers."""
        return (nB, [(l["X"].data_ptr(), l["G"].data_ptr()) for l in layers if l["kind"] == "layernorm"])

    @staticmethod
    def _dense_dims(key):
        """(B, T, d_in, d_out) of a group of dense layers from its key, whose first entries are the shapes of A and G."""
        (B, T, d_in), sG = key[0], key[1]
        if tuple(sG[:-1]) != (B, T):
            raise ValueError("A [B,T,d_in] and G [B,T,d_out] expected")
        return B, T, d_in, sG[-1]

    def _norms(self, layers):
        """(B, the norms of a micro-batch of B examples).  Refuses more examples than there are norms, and kept LayerNorm gradients, for."""
        nB, most = layers[0]["G"].shape[0], min(self.max_batch, self.sqnorms.shape[0])
        if nB > most:
            raise ValueError(f"a micro-batch of {nB} examples: the buffers hold {most}")
        return nB, self.sqnorms[:nB]

    def _check_layers(self, layers):
        """The same for every layer (the extension takes layers of one batch size only)."""
        most = max(l["G"].shape[0] for l in layers)
        if most > min(self.max_batch, self.sqnorms.shape[0]):
            raise ValueError(f"a layer of {most} examples: the buffers hold {min(self.max_batch, self.sqnorms.shape[0])}")

    def pass1(self, layers, path=B_.DP_PATH_AUTO, batch_dense=True):
        """Per-example squared global norms of one micro-batch: sqnorms[:B] = sum over all layers.  The norm is a sum
        over layers, so dense layers of one shape, and LayerNorms of one shape, are handed over together (by address: a small
        micro-batch is over on the GPU before Python has looked at 96 tensors twice)."""
        ctx = self.ctx
        nB, n = self._norms(layers)
        ctx.zero_f32(n)
        if batch_dense and path == B_.DP_PATH_AUTO and type(ctx) is B_.Context:
            # the walk below in C++ (None: something it does not expect, nothing has been called)
            done = B_._native.pass1(ctx.handle, layers, n, self.ln_keep, self._keep_buffer, self.max_batch)
            if done is not None:
                self._kept_for = None
                if type(done) is tuple:
                    B_._check(ctx.handle, *done)
                self._kept_for = done or None
                return n
        self._check_layers(layers)
        groups, ln_groups = {}, {}
        for k, l in enumerate(layers):
            kind = l["kind"]
            if kind == "dense":
                A, G = l["A"], l["G"]
                if batch_dense:
                    groups.setdefault((A.shape, G.shape, A.dtype, bool(l["has_bias"])), []).append((A.data_ptr(), G.data_ptr(), G.dtype))
                else:
                    ctx.sqnorms_dense(A, G, l["has_bias"], path, n)
            elif kind == "layernorm":
                if batch_dense:
                    ln_groups.setdefault((l["X"].shape, l["X"].dtype), []).append(k)
                else:
                    ctx.sqnorms_layernorm(l["X"], l["G"], n)
            elif kind == "tied_embedding":   # lookup table that is also the output projection; G = dY
                ctx.sqnorms_tied_embedding(l["ids"], l["G"], l["H"], l["dL"], n)
            else:
                ctx.sqnorms_embedding(l["ids"], l["G"], l["V"], l["distinct"], n)
        self._kept_for = None
        for sel in ln_groups.values():
            Xs, Gs = [layers[k]["X"] for k in sel], [layers[k]["G"] for k in sel]
            d = Xs[0].shape[-1]
            if d % 4 == 0:
                ctx.sqnorms_layernorm_keep(Xs, Gs, n, [self._keep_buffer(k, d) for k in sel])
            else:
                ctx.sqnorms_layernorm_batched(Xs, Gs, n)
        if ln_groups and all(k[0][-1] % 4 == 0 for k in ln_groups):
            self._kept_for = self._ln_token(layers, nB)
        for key, ls in groups.items():
            dims, dt = self._dense_dims(key), B_._dtype_code(key[2])
            rest = ls
            if path == B_.DP_PATH_AUTO:
                # layers reading the very same input tensor (query / key / value projections) share its Gram matrix
                by_input = {}
                for a, g, g_dt in ls:
                    by_input.setdefault(a, []).append((g, g_dt))
                shared = {a: gs for a, gs in by_input.items() if len(gs) in (2, 3)}
                if any(g_dt != key[2] for gs in shared.values() for _, g_dt in gs):
                    raise ValueError("all layers of a call must share one shape and dtype")
                for width in (3, 2):
                    sel = [(a, gs) for a, gs in shared.items() if len(gs) == width]
                    if sel:
                        B_._sqnorms_dense_shared_ptrs(ctx.handle, [a for a, _ in sel], width, [g for _, gs in sel for g, _ in gs], dt, dims,
                                                      key[3], n)
                if shared:
                    rest = [x for x in ls if x[0] not in shared]
            if rest:
                B_._sqnorms_dense_ptrs(ctx.handle, [x[0] for x in rest], [x[1] for x in rest], dt, dims, key[3], path, n)
        return n

    def pass2(self, layers, C, batch_dense=True):
        """S += sum_i clip(grad_i, C) for one micro-batch, using the norms left by pass1.  The sums of different
        layers are independent, so dense layers of one shape are handed over together (the library cuts them into launches that fill the chip)."""
        ctx = self.ctx
        nB, n = self._norms(layers)
        S = B_._f32(self.S)
        if self.S.numel() < self.P or not self.S.is_contiguous():
            raise ValueError("S must be a contiguous buffer of all parameters")
        if batch_dense and type(ctx) is B_.Context:
            done = B_._native.pass2(ctx.handle, layers, C, n, self.S, self._spans, self.ln_keep, self._kept_for, self.max_batch)
            if done is not None:
                if type(done) is tuple:
                    B_._check(ctx.handle, *done)
                return
        self._check_layers(layers)
        groups, ln_groups = {}, {}
        for k, l in enumerate(layers):
            kind = l["kind"]
            if kind == "dense":
                A, G = l["A"], l["G"]
                if batch_dense:
                    at = self._at[k]
                    groups.setdefault((A.shape, G.shape, A.dtype), []).append(
                        (A.data_ptr(), G.data_ptr(), S + at[0], S + at[1] if l["has_bias"] else None))
                else:
                    sb = self.view(self.S, k, 1) if l["has_bias"] else None
                    ctx.clip_accumulate_dense(A, G, C, n, self.view(self.S, k, 0), sb)
            elif kind == "layernorm":
                if batch_dense:
                    ln_groups.setdefault((l["X"].shape, l["X"].dtype), []).append(k)
                else:
                    ctx.clip_accumulate_layernorm(l["X"], l["G"], C, n, self.view(self.S, k, 0), self.view(self.S, k, 1))
            elif kind == "tied_embedding":
                ctx.clip_accumulate_tied_embedding(l["ids"], l["G"], l["H"], l["dL"], C, n, self.view(self.S, k, 0))
            elif l.get("distinct"):
                ctx.clip_accumulate_positions(l["G"], C, n, self.view(self.S, k, 0))   # position ids: no sort needed
            else:
                ctx.clip_accumulate_embedding(l["ids"], l["G"], l["V"], C, n, self.view(self.S, k, 0))
        kept = self._kept_for is not None and self._kept_for == self._ln_token(layers, nB)   # pass 1 of this very micro-batch left the LayerNorm gradients behind
        for sel in ln_groups.values():
            sg, sb = [S + self._at[k][0] for k in sel], [S + self._at[k][1] for k in sel]
            if kept:
                d = layers[sel[0]]["X"].shape[-1]
                ctx.clip_accumulate_layernorm_kept([self.ln_keep[k] for k in sel], nB, d, C, n, sg, sb)
            else:
                ctx.clip_accumulate_layernorm_batched([layers[k]["X"] for k in sel], [layers[k]["G"] for k in sel], C, n, sg, sb)
        for key, ls in groups.items():
            As, Gs, Ws, bs = (list(col) for col in zip(*ls))
            B_._clip_accumulate_dense_ptrs(ctx.handle, As, Gs, B_._dtype_code(key[2]), self._dense_dims(key), C, n, Ws, bs)

    def update(self, *, sigma, C, seed, step, batch_size, lr, beta1, beta2, eps=1e-11, weight_decay, zero_sum=True,
               snr_sq=None):
        """Noise + Adam over the whole flat parameter space.  With `snr_sq` (a device tensor of two floats) the
        squared norms of the aggregated gradient and of the noise vector are written there (gradient-SNR terms)."""
        kw = dict(sigma=sigma, C=C, seed=seed, step=step, batch_size=batch_size, lr=lr, beta1=beta1, beta2=beta2, eps=eps,
                  weight_decay=weight_decay, zero_sum=zero_sum)
        if snr_sq is None:
            self.ctx.noise_adamw(self.theta, self.m, self.v, self.S, **kw)
        else:
            self.ctx.zero_f32(snr_sq, 2)
            self.ctx.noise_adamw_snr(self.theta, self.m, self.v, self.S, snr_sq, **kw)
