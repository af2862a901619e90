"""Timed cases of the DP-SGD path: what a training program asks of the library, through its public entry points.

A case is a dict of plain values; `kind` says which calls one pass makes:

  step       one micro-batch through StepRunner: norms of every layer, clip-weighted sums of every layer and, with
             `update`, the noise + Adam step over all parameters (`blocks` = 0: a single dense layer hidden x ffn)
  dense      `layers` same-shaped dense layers in one call: their norms, their clip-weighted sums, or both
  embedding  the token table: norms, then the clip-weighted scatter
  tied       a table that is also the output projection of `slots` prediction slots per example: norms, then sums
  update     noise + Adam with decoupled weight decay over n parameters, with or without the gradient-SNR terms

The listed sizes are the shapes of this repository's workloads (one fp32 layer; BERT-Base- and BERT-Large-shaped
stacks, T = 128 and 512, Zipf(1.1) token ids, 20 prediction slots) and sizes next to them that a program meets as
well: a micro-batch of a few examples, sequences that are no multiple of 64, a head on 20 rows per example.
"""
import math

import torch

import paper_2108_01624_amd as dp

DEV = "cuda:0"
C = 1.0  # clip norm
ADAM = dict(beta1=0.9, beta2=0.999, lr=1e-3, weight_decay=0.5)
SIGMA, NOISE_SEED, FIRST_STEP = 0.6, 1234, 1000
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # the smallest program: one fp32 layer, whole step; launches and latency are all there is to it
        dict(name="single_layer_f32", kind="step", blocks=0, hidden=64, ffn=64, vocab=0, types=0, slots=0, batch=32, tokens=16,
             dtype="f32", update=True),
        # gradient accumulation with a micro-batch of eight: what is left per micro-batch when memory is short
        dict(name="base_microbatch", kind="step", blocks=12, hidden=768, ffn=3072, vocab=0, types=0, slots=0, batch=8, tokens=128,
             dtype="bf16", update=False),
        # a whole BERT-Large-shaped step, embedding stage included: the workload of the benchmark at half its batch
        dict(name="large_step", kind="step", blocks=24, hidden=1024, ffn=4096, vocab=30522, types=2, slots=0, batch=256, tokens=128,
             dtype="bf16", update=True),
        # norms of the attention projections of four blocks
        dict(name="norms_attention", kind="dense", passes="norms", layers=16, batch=512, tokens=128, d_in=1024, d_out=1024, dtype="bf16"),
        # norms of feed-forward layers on long sequences
        dict(name="norms_long", kind="dense", passes="norms", layers=8, batch=64, tokens=512, d_in=1024, d_out=4096, dtype="bf16"),
        # clip-weighted sums of feed-forward layers: where most of a step's time goes
        dict(name="sums_ffn", kind="dense", passes="sums", layers=4, batch=512, tokens=128, d_in=1024, d_out=4096, dtype="bf16"),
        # the same for sequences cut at 100 tokens
        dict(name="sums_ragged", kind="dense", passes="sums", layers=4, batch=96, tokens=100, d_in=768, d_out=3072, dtype="bf16"),
        # an fp32 program (inputs are not rounded to bf16): one projection, both passes
        dict(name="dense_f32", kind="dense", passes="both", layers=1, batch=16, tokens=128, d_in=768, d_out=768, dtype="f32"),
        # the transform layer of the masked-token head: 20 prediction slots per example
        dict(name="head_rows", kind="dense", passes="both", layers=1, batch=512, tokens=20, d_in=1024, d_out=1024, dtype="bf16"),
        # the word-piece table
        dict(name="token_table", kind="embedding", batch=512, tokens=128, width=1024, vocab=30522, dtype="bf16"),
        # the word-piece table when it is the output projection too
        dict(name="tied_table", kind="tied", batch=256, tokens=128, slots=20, width=1024, vocab=30528, dtype="bf16"),
        # the update of a BERT-Large-shaped model
        dict(name="update_large", kind="update", n=334088192, snr=False),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _width(rng, lo, hi):
    """A layer width: mostly a multiple of 64, now and then only of 8."""
    w = _log_int(rng, lo, hi)
    q = 64 if rng.random() < 0.75 else 8
    return max(q, w // q * q)


def draw(rng):
    kind = rng.choice(["step", "step", "dense", "dense", "dense", "embedding", "tied", "update"])
    if kind == "update":
        return dict(kind=kind, n=_log_int(rng, 1000, 334088192), snr=rng.random() < 0.5)
    if kind == "dense":
        f32 = rng.random() < 0.25
        passes = rng.choice(["norms", "sums", "both"])
        c = dict(kind=kind, passes=passes, layers=1 if f32 else rng.choice([1, 2, 4, 8, 12, 16]), batch=_log_int(rng, 4, 512),
                 tokens=_log_int(rng, 8, 192 if f32 else 640), d_in=_width(rng, 64, 1024 if f32 else 4096),
                 d_out=_width(rng, 64, 1024 if f32 else 4096), dtype="f32" if f32 else "bf16")
        while c["batch"] * c["tokens"] > (4096 if f32 else 65536) or _flops_dense(c) > (4e9 if f32 else 3e12):
            c["batch"] = (c["batch"] + 1) // 2
        return c
    if kind == "embedding":
        c = dict(kind=kind, batch=_log_int(rng, 4, 512), tokens=_log_int(rng, 16, 512), width=_width(rng, 64, 1024),
                 vocab=_log_int(rng, 512, 30522), dtype="bf16")
    elif kind == "tied":
        c = dict(kind=kind, batch=_log_int(rng, 8, 256), tokens=_log_int(rng, 16, 512), slots=rng.randint(4, 80),
                 width=_width(rng, 64, 1024), vocab=_log_int(rng, 512, 30528) // 8 * 8, dtype="bf16")
        while c["batch"] * c["slots"] > 6144:
            c["batch"] = (c["batch"] + 1) // 2
    else:
        hidden = 64 * rng.randint(2, 16)
        c = dict(kind=kind, blocks=rng.randint(1, 12), hidden=hidden, ffn=4 * hidden, vocab=rng.choice([0, _log_int(rng, 512, 30522)]),
                 types=0, slots=0, batch=_log_int(rng, 2, 256), tokens=_log_int(rng, 16, 512), dtype="bf16", update=rng.random() < 0.5)
        if c["vocab"]:
            c["types"] = 2
    while c["batch"] * c["tokens"] > 32768 * (2 if kind != "step" else 1):
        c["batch"] = (c["batch"] + 1) // 2
    return c


# ---------------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------------
class Spec:
    """One layer of a manifest as StepRunner takes it: its parameter tensors, in order."""

    def __init__(self, kind, d_in, d_out, **more):
        self.kind, self.d_in, self.d_out, self.more = kind, d_in, d_out, more

    def tensors(self):
        if self.kind == "dense":
            return [("W", (self.d_in, self.d_out))] + ([("b", (self.d_out,))] if self.more["has_bias"] else [])
        if self.kind == "layernorm":
            return [("gamma", (self.d_out,)), ("beta", (self.d_out,))]
        return [("E", (self.d_in, self.d_out))]


def _manifest(c):
    h, f = c["hidden"], c["ffn"]
    if not c["blocks"]:
        return [Spec("dense", h, f, has_bias=False)]
    m = []
    if c["vocab"]:
        m += [Spec("embedding", c["vocab"], h, ids="zipf"), Spec("embedding", 512, h, ids="position")]
    if c["types"]:
        m += [Spec("embedding", c["types"], h, ids="segment"), Spec("layernorm", 0, h)]
    for _ in range(c["blocks"]):
        m += [Spec("dense", h, h, has_bias=True) for _ in range(4)] + [Spec("layernorm", 0, h)]
        m += [Spec("dense", h, f, has_bias=True), Spec("dense", f, h, has_bias=True), Spec("layernorm", 0, h)]
    return m


class Draws:
    """Seeded draws on the GPU."""

    def __init__(self, seed, dtype="f32"):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(int(seed))
        self.dtype = DTYPES[dtype]

    def normal(self, shape, std=1.0, scale=None):
        """N(0, std^2), example i multiplied by scale[i]; drawn in fp32 piece by piece, rounded to the case's type."""
        out = torch.empty(shape, dtype=self.dtype, device=DEV)
        per = max(1, (1 << 27) // max(1, math.prod(shape[1:])))
        for r in range(0, shape[0], per):
            x = torch.randn((min(per, shape[0] - r),) + tuple(shape[1:]), generator=self.gen, device=DEV).mul_(std)
            out[r:r + per] = x if scale is None else x * scale[r:r + per].view((-1,) + (1,) * (len(shape) - 1))
        return out

    def uniform(self, shape):
        return torch.rand(shape, generator=self.gen, device=DEV)

    def scales(self, batch):
        """Per-example gradient scales, log-uniform over [1e-4, 1]: some examples stay under the clip norm."""
        return torch.exp(self.uniform((batch,)) * math.log(1e4)) * 1e-4

    def zipf(self, batch, tokens, vocab):
        w = torch.arange(1, vocab + 1, dtype=torch.float64, device=DEV) ** -1.1
        cdf = torch.cumsum(w, 0) / w.sum()
        u = torch.rand((batch, tokens), generator=self.gen, device=DEV, dtype=torch.float64)
        return torch.searchsorted(cdf, u).clamp_(max=vocab - 1).to(torch.int32)

    def sqnorms(self, batch):
        """Finished squared norms, log-uniform over [C^2 / 100, 100 C^2]."""
        return torch.exp((self.uniform((batch,)) * 2 - 1) * math.log(100.0)) * (C * C)


_ctx = None


def _context():
    """The one context a program keeps: its stream and workspace."""
    global _ctx
    if _ctx is None:
        _ctx = dp.Context()
    return _ctx


def _step_inputs(c, seed):
    """(manifest, layer inputs) of one micro-batch."""
    r, man, B, T = Draws(seed, c["dtype"]), _manifest(c), c["batch"], c["tokens"]
    scale, layers, shared = r.scales(B), [], None
    for s in man:
        l = dict(kind=s.kind)
        if s.kind == "embedding":
            # the three tables are summed: one upstream gradient for all of them
            shared = r.normal((B, T, s.d_out), 1e-2, scale) if shared is None else shared
            how = s.more["ids"]
            if how == "zipf":
                ids = r.zipf(B, T, s.d_in)
            else:
                row = torch.arange(T, dtype=torch.int32, device=DEV)
                ids = (row if how == "position" else (row >= (T + 1) // 2).to(torch.int32)).expand(B, T).contiguous()
            l.update(ids=ids, G=shared, V=s.d_in, distinct=how == "position")
        elif s.kind == "layernorm":
            l.update(X=r.normal((B, T, s.d_out)), G=r.normal((B, T, s.d_out), 1e-2, scale))
        else:
            l.update(A=r.normal((B, T, s.d_in)), G=r.normal((B, T, s.d_out), 1e-2, scale), has_bias=s.more["has_bias"])
        layers.append(l)
    return man, layers


def _moments(c, seed, n):
    """theta, m, v of a run under way: gradients there are mostly noise of standard deviation sigma C / |B_t|."""
    r = Draws(seed + 77)
    g = SIGMA * C / c.get("batch", 65536)
    return r.normal((n,), 0.02), r.normal((n,), 0.2 * g), (r.uniform((n,)) + 0.5) * (g * g)


def _tied_inputs(c, seed):
    """ids, dY, H, dL: logit gradients are dense and small with one large entry per used slot (the label's)."""
    r, B, T, M, d, V = Draws(seed, c["dtype"]), c["batch"], c["tokens"], c["slots"], c["width"], c["vocab"]
    scale = r.scales(B)
    ids, dY, H = r.zipf(B, T, V), r.normal((B, T, d), 1e-2, scale), r.normal((B, M, d))
    dL = r.normal((B, M, V), 1e-2 / 8, scale)
    labels = r.zipf(B, M, V).long()
    dL.scatter_(2, labels[:, :, None], (-8e-2 * scale[:, None, None]).expand(B, M, 1).to(dL.dtype))
    used = torch.arange(M, device=DEV)[None, :] < ((1 + r.uniform((B,))) * 0.5 * M).ceil()[:, None]
    return ids, dY, H, dL.mul_(used[:, :, None].to(dL.dtype))


def prepare(case, seed):
    c, ctx = case, _context()
    st = dict(case=c, ctx=ctx)
    if c["kind"] == "step":
        man, layers = _step_inputs(c, seed)
        run = dp.StepRunner(ctx, man, c["batch"], device=DEV)
        if c["update"]:
            for buf, x in zip((run.theta, run.m, run.v), _moments(c, seed, run.P)):
                buf.copy_(x)
        st.update(layers=layers, runner=run, t=FIRST_STEP)
        return st
    if c["kind"] == "update":
        theta, m, v = _moments(c, seed, c["n"])
        st.update(theta=theta, m=m, v=v, S=Draws(seed + 78).normal((c["n"],), 0.5), t=FIRST_STEP,
                  snr=torch.zeros(2, dtype=torch.float32, device=DEV))
        return st
    B = c["batch"]
    if c["kind"] == "dense":
        r, L, T = Draws(seed, c["dtype"]), c["layers"], c["tokens"]
        scale = r.scales(B)
        st.update(A=[r.normal((B, T, c["d_in"])) for _ in range(L)], G=[r.normal((B, T, c["d_out"]), 1e-2, scale) for _ in range(L)])
        if c["passes"] != "norms":
            st.update(W=[torch.zeros(c["d_in"], c["d_out"], device=DEV) for _ in range(L)],
                      b=[torch.zeros(c["d_out"], device=DEV) for _ in range(L)])
        st["n"] = r.sqnorms(B) if c["passes"] == "sums" else torch.zeros(B, device=DEV)
    elif c["kind"] == "embedding":
        r = Draws(seed, c["dtype"])
        st.update(ids=r.zipf(B, c["tokens"], c["vocab"]), G=r.normal((B, c["tokens"], c["width"]), 1e-2, r.scales(B)))
    else:
        st["in"] = _tied_inputs(c, seed)
    if c["kind"] in ("embedding", "tied"):
        st.update(n=torch.zeros(B, device=DEV), E=torch.zeros(c["vocab"], c["width"], device=DEV))
    return st


# ---------------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------------
def run(st):
    c, ctx = st["case"], st["ctx"]
    if c["kind"] == "step":
        r = st["runner"]
        n = r.pass1(st["layers"])
        r.pass2(st["layers"], C)
        if not c["update"]:
            return dict(sqnorms=n, sums=r.S)  # the next micro-batch of the mega-batch adds to the same sums
        r.update(sigma=SIGMA, C=C, seed=NOISE_SEED, step=st["t"], batch_size=c["batch"], **ADAM)
        st["t"] += 1
        return dict(sqnorms=n, theta=r.theta, m=r.m, v=r.v)
    if c["kind"] == "update":
        kw = dict(sigma=SIGMA, C=C, seed=NOISE_SEED, step=st["t"], batch_size=65536, zero_sum=True, **ADAM)
        st["t"] += 1
        if c["snr"]:
            ctx.zero_f32(st["snr"])
            ctx.noise_adamw_snr(st["theta"], st["m"], st["v"], st["S"], st["snr"], **kw)
            return dict(theta=st["theta"], m=st["m"], v=st["v"], sums=st["S"], snr=st["snr"])
        ctx.noise_adamw(st["theta"], st["m"], st["v"], st["S"], **kw)
        return dict(theta=st["theta"], m=st["m"], v=st["v"], sums=st["S"])
    n = st["n"]
    if c["kind"] == "dense":
        if c["passes"] != "sums":
            ctx.zero_f32(n)
            ctx.sqnorms_dense_batched(st["A"], st["G"], True, dp.DP_PATH_AUTO, n)
        if c["passes"] == "norms":
            return dict(sqnorms=n)
        ctx.clip_accumulate_dense_batched(st["A"], st["G"], C, n, st["W"], st["b"])
        return dict(W=st["W"], b=st["b"], sqnorms=n)
    ctx.zero_f32(n)
    if c["kind"] == "embedding":
        ctx.sqnorms_embedding(st["ids"], st["G"], c["vocab"], False, n)
        ctx.clip_accumulate_embedding(st["ids"], st["G"], c["vocab"], C, n, st["E"])
    else:
        ctx.sqnorms_tied_embedding(*st["in"], n)
        ctx.clip_accumulate_tied_embedding(*st["in"], C, n, st["E"])
    return dict(sqnorms=n, E=st["E"])


# ---------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------------
def _norm_flops(T, d_in, d_out):
    """Per example: the symmetric Gram form or the materialised gradient, whichever is less."""
    return min(1.0 * T * (T + 1) * (d_in + d_out), 2.0 * T * d_in * d_out)


def _flops_dense(c):
    f = 0.0
    if c["passes"] != "sums":
        f += _norm_flops(c["tokens"], c["d_in"], c["d_out"])
    if c["passes"] != "norms":
        f += 2.0 * c["tokens"] * c["d_in"] * c["d_out"]
    return c["layers"] * c["batch"] * f


def work(case):
    c = case
    if c["kind"] == "update":
        return dict(bytes=32.0 * c["n"], flops=100.0 * c["n"])
    rows, E = c["batch"] * c["tokens"], 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "dense":
        b = c["layers"] * rows * (c["d_in"] + c["d_out"]) * E
        if c["passes"] != "norms":
            b += 8.0 * c["layers"] * (c["d_in"] + 1) * c["d_out"]
        return dict(bytes=b, flops=_flops_dense(c))
    if c["kind"] == "embedding":
        # sums: the rows of the tokens that occur, read and written
        return dict(bytes=rows * (c["width"] * E + 4) + 8.0 * min(rows // 6, c["vocab"]) * c["width"], flops=6.0 * rows * c["width"])
    if c["kind"] == "tied":
        M, d, V, B, T = c["slots"], c["width"], c["vocab"], c["batch"], c["tokens"]
        return dict(bytes=E * (rows * d + B * M * (d + V)) + 4 * rows + 8.0 * V * d,
                    flops=2.0 * B * M * V * d + B * _norm_flops(M, V, d) + 2.0 * rows * M * d)
    by = fl = P = 0.0
    seen = False
    for s in _manifest(c):
        P += sum(math.prod(shape) for _, shape in s.tensors())
        if s.kind == "dense":
            by += rows * (s.d_in + s.d_out) * E
            fl += 2.0 * rows * s.d_in * s.d_out + c["batch"] * _norm_flops(c["tokens"], s.d_in, s.d_out)
        elif s.kind == "layernorm":
            by += rows * 2 * s.d_out * E
            fl += 8.0 * rows * s.d_out
        else:
            by += rows * 4 + (0 if seen else rows * s.d_out * E)
            fl += 6.0 * rows * s.d_out
            seen = True
    return dict(bytes=by + (24.0 if c["update"] else 8.0) * P, flops=fl + (100.0 * P if c["update"] else 0.0))


def tolerance(case):
    """About four times what two correct implementations differ by.  fp32 sums in another order: below 3e-6 in the 2-norm.
    bf16 dense sums may also round c * g to bf16 once (2^-9 per term, averaged over the sum), which the interface allows
    for row counts per example and widths that are no multiples of its tiles: 1.7e-3."""
    c = case
    if c["kind"] == "update" or (c["kind"] == "step" and c["update"]):
        return dict(rel=1e-5, max=1e-2)
    if c["dtype"] == "f32" or c["kind"] == "embedding" or (c["kind"] == "dense" and c["passes"] == "norms"):
        return dict(rel=1e-5, max=1e-3)
    return dict(rel=7e-3, max=7e-2)


# ---------------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------------------------------
def _gram_norms(A, G, bias):
    out = []
    per = max(1, (1 << 27) // (A.shape[1] * max(A.shape[2], G.shape[2], A.shape[1])))
    for i in range(0, A.shape[0], per):
        a, g = A[i:i + per].double(), G[i:i + per].double()
        aa, gg = (torch.matmul(x, x.transpose(1, 2).contiguous()) for x in (a, g))
        out.append(((aa + (1.0 if bias else 0.0)) * gg).sum((1, 2)))
    return torch.cat(out)


def _factors(n):
    return torch.where(n > 0, (C / n.clamp(min=1e-300).sqrt()).clamp(max=1.0), torch.ones_like(n))


def _scatter_norms(ids, G, vocab):
    B, T, d = G.shape
    key, where = torch.unique(ids.long() + vocab * torch.arange(B, device=DEV)[:, None], return_inverse=True)
    rows = torch.zeros(key.numel(), d, dtype=torch.float64, device=DEV).index_add_(0, where.reshape(-1), G.reshape(-1, d).double())
    return torch.zeros(B, dtype=torch.float64, device=DEV).index_add_(0, key // vocab, rows.square().sum(1))


def _weighted(G, c):
    return G.double() * c[:, None, None]


def _scatter_sums(ids, G, vocab, c):
    d = G.shape[-1]
    out = torch.zeros(vocab, d, dtype=torch.float64, device=DEV)
    return out.index_add_(0, ids.reshape(-1).long(), _weighted(G, c).reshape(-1, d))


def _dense_sums(A, G, c):
    g = _weighted(G, c).reshape(-1, G.shape[-1])
    at = A.reshape(-1, A.shape[-1]).t().contiguous().double()
    return torch.matmul(at, g), g.sum(0)


def _normals(n, seed, step):
    """The standard normals of elements 0 .. n-1: Philox4x32-10 words, Box-Muller on the word pairs (0, 1) and (2, 3)."""
    mask = 0xFFFFFFFF
    out = torch.empty(n, dtype=torch.float64, device=DEV)
    for b0 in range(0, (n + 3) // 4, 1 << 23):
        blk = torch.arange(b0, min(b0 + (1 << 23), (n + 3) // 4), dtype=torch.int64, device=DEV)
        w = [blk & mask, blk >> 32, torch.full_like(blk, step & mask), torch.full_like(blk, step >> 32)]
        k0, k1 = seed & mask, seed >> 32
        for _ in range(10):
            p, q = w[0] * 0xD2511F53, w[2] * 0xCD9E8D57
            w = [((q >> 32) & mask) ^ w[1] ^ k0, q & mask, ((p >> 32) & mask) ^ w[3] ^ k1, p & mask]
            k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
        u = [((x >> 9).double() + 0.5) * 2.0 ** -23 for x in w]
        z = []
        for a, b in ((u[0], u[1]), (u[2], u[3])):
            rho = torch.sqrt(-2.0 * torch.log(a))
            z += [rho * torch.cos(2 * math.pi * b), rho * torch.sin(2 * math.pi * b)]
        z = torch.stack(z, 1).reshape(-1)
        out[4 * b0:4 * b0 + z.numel()] = z[:n - 4 * b0]
    return out


def _adam(theta, m, v, S, batch_size):
    """theta, m, v after one update, and the noise vector (the scalars as fp32 holds them)."""
    f = lambda x: float(torch.tensor(x, dtype=torch.float32))  # noqa: E731
    b1, b2 = f(ADAM["beta1"]), f(ADAM["beta2"])
    noise = _normals(S.numel(), NOISE_SEED, FIRST_STEP) * (f(SIGMA) * f(C))
    g = (S.double() + noise) / batch_size
    m = b1 * m.double() + (1 - b1) * g
    v = b2 * v.double() + (1 - b2) * g * g
    mh, vh = m / (1 - b1 ** FIRST_STEP), v / (1 - b2 ** FIRST_STEP)
    theta = theta.double()
    return theta - f(ADAM["lr"]) * (mh / (vh.sqrt() + 1e-11) + f(ADAM["weight_decay"]) * theta), m, v, noise


def _exact_step(c, seed):
    man, layers = _step_inputs(c, seed)
    n = torch.zeros(c["batch"], dtype=torch.float64, device=DEV)
    for s, l in zip(man, layers):
        if s.kind == "dense":
            n += _gram_norms(l["A"], l["G"], l["has_bias"])
        elif s.kind == "layernorm":
            n += (l["X"].double() * l["G"].double()).sum(1).square().sum(1) + l["G"].double().sum(1).square().sum(1)
        else:
            n += _scatter_norms(l["ids"], l["G"], l["V"])
    cf, sums = _factors(n), []
    for s, l in zip(man, layers):
        if s.kind == "dense":
            w, b = _dense_sums(l["A"], l["G"], cf)
            sums += [w.reshape(-1)] + ([b] if l["has_bias"] else [])
        elif s.kind == "layernorm":
            g = _weighted(l["G"], cf)
            sums += [(g * l["X"].double()).sum((0, 1)), g.sum((0, 1))]
        else:
            sums.append(_scatter_sums(l["ids"], l["G"], l["V"], cf).reshape(-1))
    S = torch.cat(sums)
    if not c["update"]:
        return dict(sqnorms=n, sums=S)
    theta, m, v, _ = _adam(*_moments(c, seed, S.numel()), S, c["batch"])
    return dict(sqnorms=n, theta=theta, m=m, v=v)


def exact(case, seed):
    c = case
    if c["kind"] == "step":
        return _exact_step(c, seed)
    st = prepare(c, seed)
    if c["kind"] == "update":
        theta, m, v, noise = _adam(st["theta"], st["m"], st["v"], st["S"], 65536)
        out = dict(theta=theta, m=m, v=v, sums=torch.zeros(c["n"], dtype=torch.float64, device=DEV))
        if c["snr"]:
            out["snr"] = torch.stack([st["S"].double().square().sum(), noise.square().sum()])
        return out
    if c["kind"] == "dense":
        n = st["n"].double()
        if c["passes"] != "sums":
            n = sum(_gram_norms(a, g, True) for a, g in zip(st["A"], st["G"]))
        if c["passes"] == "norms":
            return dict(sqnorms=n)
        both = [_dense_sums(a, g, _factors(n)) for a, g in zip(st["A"], st["G"])]
        return dict(W=[w for w, _ in both], b=[b for _, b in both], sqnorms=n)
    if c["kind"] == "embedding":
        n = _scatter_norms(st["ids"], st["G"], c["vocab"])
        return dict(sqnorms=n, E=_scatter_sums(st["ids"], st["G"], c["vocab"], _factors(n)))
    ids, dY, H, dL = st["in"]
    n = _scatter_norms(ids, dY, c["vocab"]) + _gram_norms(dL, H, False)
    at = torch.gather(dL, 2, ids.long()[:, None, :].expand(-1, c["slots"], -1)).double()
    n = n + 2 * (at * torch.matmul(H.double(), dY.double().transpose(1, 2).contiguous())).sum((1, 2))
    cf = _factors(n)
    return dict(sqnorms=n, E=_scatter_sums(ids, dY, c["vocab"], cf) + _dense_sums(dL, H, cf)[0])
