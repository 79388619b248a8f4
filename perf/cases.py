"""The work by which this library's speed is judged: what training and inference programs ask of it.

A case is a dict of plain values.  `path` says which public entry points it goes through:
  layer    one SVD-decomposed linear layer: forward, and for direction "train" its backward, with the
           freeze mask, bias and optimizer step that the case states;
  stack    the FFN stack of a network (linear, GELU, linear per block), forward and two-part backward;
  encoder  the decomposed linears of a transformer encoder (Q/K/V group, output projection, FFN), the same way;
  conv     one Tucker-decomposed convolution, forward or forward and backward.
Factors are drawn directly at N(0, 1/r) and N(0, 1/in): speed and arithmetic do not depend on how they
were obtained.  Buffers that a program keeps from step to step (results, workspace) belong to the state.
"""
import torch

from paper_2309_03824_amd import binding as lrd

BF, F32 = torch.bfloat16, torch.float32
SGD = (1e-4, 0.9, 1e-4)         # learning rate, momentum, weight decay


def listed():
    return [
        # Serving one short sequence: the FFN up-projection of the encoder, forward only.  Latency counts.
        dict(name="infer_short", path="layer", direction="infer", dtype="bf16", tokens=48, n_in=1024, n_out=4096, rank=256, mask=0,
             bias=True, update=False),
        # The single fp32 layer (768 x 768, rank 200 quantized to 208, first factor frozen).
        dict(name="layer_f32", path="layer", direction="train", dtype="f32", tokens=256, n_in=768, n_out=768, rank=208, mask=1,
             bias=False, update=False),
        # Fine-tuning with a small batch: nothing frozen yet, bias trained.
        dict(name="layer_small_batch", path="layer", direction="train", dtype="bf16", tokens=509, n_in=768, n_out=3072, rank=192, mask=0,
             bias=True, update=False),
        # A rank straight from a compression ratio, before quantization, nothing frozen, and a ragged batch.
        dict(name="layer_raw_rank", path="layer", direction="train", dtype="bf16", tokens=4100, n_in=1024, n_out=4096, rank=257, mask=0,
             bias=True, update=False),
        # The large layer of the rank sweep, first factor frozen.
        dict(name="layer_4096", path="layer", direction="train", dtype="bf16", tokens=16384, n_in=4096, n_out=4096, rank=512, mask=1,
             bias=False, update=False),
        # A training step of one FFN down-projection with the optimizer in the backward, second factor frozen.
        dict(name="layer_update", path="layer", direction="train", dtype="bf16", tokens=8192, n_in=3072, n_out=768, rank=192, mask=2,
             bias=True, update=True),
        # The 12-block FFN stack, launched call by call.
        dict(name="ffn_stack", path="stack", layers=12, tokens=8192, width=768, ff=3072, rank=192, mask=2, graph=False),
        # The 12-layer encoder's training step, replayed from a captured graph as a training loop does.
        dict(name="encoder_step", path="encoder", layers=12, tokens=8192, width=1024, ff=4096, rank=256, mask=1, graph=True),
        # Early ResNet stage, many pixels and few channels, core frozen.
        dict(name="conv_64_core_frozen", path="conv", direction="train", images=128, size=56, c_in=64, c_out=64, r1=32, r2=32, stride=1, mask=2),
        # Later stage, the odd step of sequential freezing: 1x1 layers frozen, core trained.
        dict(name="conv_256_core_trained", path="conv", direction="train", images=128, size=14, c_in=256, c_out=256, r1=128, r2=128, stride=1, mask=5),
        # Last stage at the rank a 2x compression gives (512 channels: 309), nothing frozen.
        dict(name="conv_512_raw_rank", path="conv", direction="train", images=128, size=7, c_in=512, c_out=512, r1=309, r2=309, stride=1, mask=0),
        # Inference through a stride-2 transition, small batch.
        dict(name="conv_stride2_infer", path="conv", direction="infer", images=24, size=28, c_in=128, c_out=256, r1=64, r2=128, stride=2, mask=0),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _rank(rng, most):
    """A rank between a fifth and a half of the narrow side: quantized to 64 or 16, or as it came."""
    r = rng.randint(max(1, most // 5), most // 2)
    m = rng.choice((64, 64, 16, 1))
    return max(m, r // m * m)


def draw(rng):
    kind = rng.choice(("infer", "layer", "layer", "layer", "f32", "stack", "encoder", "conv", "conv", "conv"))
    widths = (512, 768, 1000, 1024, 1536, 2048, 3072, 4096)
    if kind == "infer":
        n_in, n_out = rng.choice(widths), rng.choice(widths)
        return dict(path="layer", direction="infer", dtype="bf16", tokens=_log(rng, 4, 4096), n_in=n_in, n_out=n_out,
                    rank=_rank(rng, min(n_in, n_out)), mask=0, bias=rng.random() < 0.7, update=False)
    if kind == "layer":
        n_in, n_out = rng.choice(widths), rng.choice(widths)
        mask = rng.choice((0, 1, 2))
        return dict(path="layer", direction="train", dtype="bf16", tokens=_log(rng, 128, 16384), n_in=n_in, n_out=n_out,
                    rank=_rank(rng, min(n_in, n_out)), mask=mask, bias=rng.random() < 0.6, update=mask != 0 and rng.random() < 0.4)
    if kind == "f32":
        n_in, n_out = rng.choice((256, 384, 768, 1000, 1024)), rng.choice((256, 384, 768, 1000, 1024))
        return dict(path="layer", direction="train", dtype="f32", tokens=_log(rng, 64, 2048), n_in=n_in, n_out=n_out,
                    rank=_rank(rng, min(n_in, n_out)), mask=rng.choice((0, 1, 2)), bias=rng.random() < 0.3, update=False)
    if kind in ("stack", "encoder"):
        width = rng.choice((512, 768, 1024))
        return dict(path=kind, layers=rng.randint(2, 6), tokens=_log(rng, 1024, 8192) // 8 * 8, width=width, ff=4 * width,
                    rank=rng.choice((width // 4, width // 4, width // 4 + 32, width // 8 * 3)), mask=rng.choice((1, 2)), graph=rng.random() < 0.5)
    c = rng.choice((64, 128, 256, 512))
    stride = rng.choice((1, 1, 2)) if c < 512 else 1
    s = c * stride
    size = max(5, 3584 // c + rng.randint(-2, 3))
    mode = rng.choice(("half", "half", "multiple", "raw"))
    r1, r2 = c // 2, s // 2
    if mode != "half":
        r1, r2 = int(c * rng.uniform(0.3, 0.7)), int(s * rng.uniform(0.3, 0.7))
    if mode == "multiple":
        r1, r2 = max(16, r1 // 16 * 16), max(16, r2 // 16 * 16)
    return dict(path="conv", direction=rng.choice(("infer", "train", "train")), images=_log(rng, 8, 128), size=size, c_in=c, c_out=s, r1=r1, r2=r2,
                stride=stride, mask=rng.choice((0, 2, 5)))


# --------------------------------------------------------------------------------------- states
class _Maker:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(self, *shape, std=1.0, dt=BF):
        return torch.randn(*shape, device="cuda", generator=self.gen).mul_(std).to(dt)

    @staticmethod
    def empty(*shape, dt=BF):
        return torch.empty(*shape, dtype=dt, device="cuda")

    def pair(self, n_out, n_in, r, dt=BF):
        return self.normal(n_out, r, std=r ** -0.5, dt=dt), self.normal(r, n_in, std=n_in ** -0.5, dt=dt)


def _workspace(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device="cuda")


class _Layer:
    def __init__(self, c, seed):
        m, dt = _Maker(seed), F32 if c["dtype"] == "f32" else BF
        code = lrd.F32 if c["dtype"] == "f32" else lrd.BF16
        T, n_in, n_out, r = c["tokens"], c["n_in"], c["n_out"], c["rank"]
        self.mask, self.train, self.update = c["mask"], c["direction"] == "train", c["update"]
        self.X = m.normal(T, n_in, dt=dt)
        self.U, self.V = m.pair(n_out, n_in, r, dt)
        self.bias = m.normal(n_out, std=0.1, dt=F32) if c["bias"] else None
        self.Y = m.empty(T, n_out, dt=dt)
        self.H = m.empty(T, r, dt=dt) if self.train else None
        nbytes = lrd.linear_workspace_bytes(T, n_in, n_out, r, code, self.mask)
        if self.train:
            tv, tu = not self.mask & lrd.FREEZE_L0, not self.mask & lrd.FREEZE_L1
            self.dY = m.normal(T, n_out, dt=dt)
            self.dX = m.empty(T, n_in, dt=dt)
            self.dbias = m.empty(n_out, dt=F32) if c["bias"] else None
            if self.update:
                nbytes = max(nbytes, lrd.linear_sgd_workspace_bytes(T, n_in, n_out, r, code, self.mask))
                self.opt = lrd.Sgd(*SGD)
                self.Vm, self.Um = (self.V.float() if tv else None), (self.U.float() if tu else None)
                self.Vs, self.Us = (torch.zeros_like(self.Vm) if tv else None), (torch.zeros_like(self.Um) if tu else None)
            else:
                self.dV, self.dU = (m.empty(r, n_in, dt=F32) if tv else None), (m.empty(n_out, r, dt=F32) if tu else None)
        self.ws = _workspace(nbytes)

    def run(self):
        lrd.linear_fwd(self.X, self.V, self.U, self.bias, self.Y, self.H, self.ws)
        if not self.train:
            return self.Y
        out = dict(Y=self.Y, H=self.H, dX=self.dX, dbias=self.dbias)
        if self.update:
            lrd.linear_bwd_sgd(self.dY, self.X, self.H, self.V, self.U, self.dX, self.Vm, self.Um, self.Vs, self.Us, self.dbias, self.mask,
                               None, lrd.ACT_NONE, self.opt, self.ws)
            return dict(out, V=self.V, U=self.U, Vm=self.Vm, Um=self.Um, Vs=self.Vs, Us=self.Us)
        lrd.linear_bwd(self.dY, self.X, self.H, self.V, self.U, self.dX, self.dV, self.dU, self.dbias, self.mask, self.ws)
        return dict(out, dV=self.dV, dU=self.dU)


class _Graphed:
    """A state whose step may be replayed from a captured graph."""

    def run(self):
        if self.graph is None:
            self.step()
        else:
            self.graph.replay()
        return self.outputs()

    def capture(self, wanted):
        self.graph = None
        if wanted:
            self.step()          # first-call set-up stays out of the capture
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                self.step()
            self.graph = graph


class _Stack(_Graphed):
    def __init__(self, c, seed):
        m = _Maker(seed)
        L, T, d, ff, r = c["layers"], c["tokens"], c["width"], c["ff"], c["rank"]
        self.L, self.mask = L, c["mask"]
        self.tv, self.tu = not self.mask & lrd.FREEZE_L0, not self.mask & lrd.FREEZE_L1
        self.up, self.dn = self._linears(m, L, T, d, ff, r), self._linears(m, L, T, ff, d, r)
        # G[l] enters block l's second layer from behind; the stack's result is G[L - 1] (loss half the squared norm)
        self.Xs, self.G = m.empty(L, T, d), m.empty(L, T, d)
        self.Xs[0].copy_(m.normal(T, d))
        self.Z, self.A, self.gZ, self.dX0 = m.empty(L, T, ff), m.empty(L, T, ff), m.empty(L, T, ff), m.empty(T, d)
        self.ws = _workspace(max(f(*a, lrd.BF16, 0) for a in ((T, d, ff, r), (T, ff, d, r)) for f in (
            lrd.linear_workspace_bytes, lambda *b: lrd.linear_wgrad_batched_workspace_bytes(L, *b))))
        self.capture(c["graph"])

    def _linears(self, m, L, T, n_in, n_out, r):
        return dict(f=[m.pair(n_out, n_in, r) for _ in range(L)], H=m.empty(L, T, r), dH=m.empty(L, T, r),
                    dU=m.empty(L, n_out, r, dt=F32) if self.tu else None, dV=m.empty(L, r, n_in, dt=F32) if self.tv else None)

    def step(self):
        up, dn, L = self.up, self.dn, self.L
        for l in range(L):
            U, V = up["f"][l]
            lrd.linear_fwd_act(self.Xs[l], V, U, None, self.Z[l], self.A[l], up["H"][l], lrd.ACT_GELU, self.ws)
            U, V = dn["f"][l]
            lrd.linear_fwd(self.A[l], V, U, None, self.Xs[l + 1] if l + 1 < L else self.G[l], dn["H"][l], self.ws)
        for l in reversed(range(L)):
            U, V = dn["f"][l]
            lrd.linear_bwd_data(self.G[l], V, U, self.gZ[l], dn["dH"][l], self.Z[l], lrd.ACT_GELU, self.ws)
            U, V = up["f"][l]
            lrd.linear_bwd_data(self.gZ[l], V, U, self.G[l - 1] if l > 0 else self.dX0, up["dH"][l], None, lrd.ACT_NONE, self.ws)
        for s, dY, X in ((dn, self.G, self.A), (up, self.gZ, self.Xs)):
            self._wgrads(s, dY, X)

    def _wgrads(self, s, dY, X):
        lrd.linear_wgrad_batched(dY if self.tu else None, s["H"] if self.tu else None, s["dH"] if self.tv else None, X if self.tv else None,
                                 s["dV"], s["dU"], self.mask, self.ws)

    def outputs(self):
        return dict(Y=self.G[self.L - 1], dX0=self.dX0, **{n + k: s[k] for n, s in (("up_", self.up), ("dn_", self.dn)) for k in ("dU", "dV")})


class _Encoder(_Stack):
    def __init__(self, c, seed):
        m = _Maker(seed)
        L, T, d, ff, r = c["layers"], c["tokens"], c["width"], c["ff"], c["rank"]
        self.L, self.mask, self.r = L, c["mask"], r
        self.tv, self.tu = not self.mask & lrd.FREEZE_L0, not self.mask & lrd.FREEZE_L1
        self.o, self.up, self.dn = self._linears(m, L, T, d, d, r), self._linears(m, L, T, d, ff, r), self._linears(m, L, T, ff, d, r)
        self.q = dict(f=[(m.normal(3, d, r, std=r ** -0.5), m.normal(3 * r, d, std=d ** -0.5)) for _ in range(L)], H=m.empty(L, T, 3 * r),
                      dH=m.empty(L, T, 3 * r), dU=m.empty(3, L, d, r, dt=F32) if self.tu else None,
                      dV=m.empty(L, 3 * r, d, dt=F32) if self.tv else None)
        # what the attention, which is not this library's, hands to the output projection and back to Q/K/V
        self.attn, self.dqkv = m.normal(L, T, d), m.normal(L, 3, T, d, std=1e-2)
        self.qkv, self.gattn = m.empty(L, 3, T, d), m.empty(L, T, d)
        self.Xo, self.gXo, self.Z, self.A, self.gZ = m.empty(L, T, d), m.empty(L, T, d), m.empty(L, T, ff), m.empty(L, T, ff), m.empty(L, T, ff)
        self.Xs, self.G, self.dX0 = m.empty(L, T, d), m.empty(L, T, d), m.empty(T, d)
        self.Xs[0].copy_(m.normal(T, d))
        self.ws = _workspace(max([lrd.linear_group_workspace_bytes(T, d, d, r, 3, lrd.BF16, 0),
                                  lrd.linear_wgrad_batched_workspace_bytes(L, T, d, d, 3 * r, lrd.BF16, 0)] +
                                 [f(*a, lrd.BF16, 0) for a in ((T, d, d, r), (T, d, ff, r), (T, ff, d, r)) for f in (
                                     lrd.linear_workspace_bytes, lambda *b: lrd.linear_wgrad_batched_workspace_bytes(L, *b))]))
        self.capture(c["graph"])

    def step(self):
        q, o, up, dn, L = self.q, self.o, self.up, self.dn, self.L
        for l in range(L):
            U, V = q["f"][l]
            lrd.linear_group_fwd(self.Xs[l], V, U, None, self.qkv[l], q["H"][l], self.ws)
            U, V = o["f"][l]
            lrd.linear_fwd(self.attn[l], V, U, None, self.Xo[l], o["H"][l], self.ws)
            U, V = up["f"][l]
            lrd.linear_fwd_act(self.Xo[l], V, U, None, self.Z[l], self.A[l], up["H"][l], lrd.ACT_GELU, self.ws)
            U, V = dn["f"][l]
            lrd.linear_fwd(self.A[l], V, U, None, self.Xs[l + 1] if l + 1 < L else self.G[l], dn["H"][l], self.ws)
        for l in reversed(range(L)):
            U, V = dn["f"][l]
            lrd.linear_bwd_data(self.G[l], V, U, self.gZ[l], dn["dH"][l], self.Z[l], lrd.ACT_GELU, self.ws)
            U, V = up["f"][l]
            lrd.linear_bwd_data(self.gZ[l], V, U, self.gXo[l], up["dH"][l], None, lrd.ACT_NONE, self.ws)
            U, V = o["f"][l]
            lrd.linear_bwd_data(self.gXo[l], V, U, self.gattn[l], o["dH"][l], None, lrd.ACT_NONE, self.ws)
            U, V = q["f"][l]
            lrd.linear_group_bwd_data(self.dqkv[l], V, U, self.G[l - 1] if l > 0 else self.dX0, q["dH"][l], self.ws)
        for s, dY, X in ((dn, self.G, self.A), (up, self.gZ, self.Xo), (o, self.gXo, self.attn)):
            self._wgrads(s, dY, X)
        if self.tv:      # the stacked first factors of a group: one gradient of depth 3 r
            lrd.linear_wgrad_batched(None, None, q["dH"], self.Xs, q["dV"], None, self.mask | 2, self.ws)
        if self.tu:      # the second factors: member g of every layer, addressed inside the stacks
            for g in range(3):
                lrd.linear_wgrad_batched(self.dqkv[:, g], q["H"][:, :, g * self.r:(g + 1) * self.r], None, None, None, q["dU"][g],
                                         self.mask | 1, self.ws)

    def outputs(self):
        out = dict(super().outputs(), qkv=self.qkv, gattn=self.gattn)
        out.update({n + k: s[k] for n, s in (("o_", self.o), ("qkv_", self.q)) for k in ("dU", "dV")})
        return out


class _Conv:
    def __init__(self, c, seed):
        m = _Maker(seed)
        N, hw, C, S, r1, r2, k = c["images"], c["size"], c["c_in"], c["c_out"], c["r1"], c["r2"], 3
        self.mask, self.train = c["mask"], c["direction"] == "train"
        self.g = lrd.conv_geom(N, hw, hw, C, S, r1, r2, k, c["stride"], 1)
        ho, wo = self.g.out_hw()
        self.X, self.Y = m.normal(N, hw, hw, C), m.empty(N, ho, wo, S)
        self.P1, self.P2 = m.normal(r1, C, std=C ** -0.5), m.normal(S, r2, std=r2 ** -0.5)
        self.G = m.normal(r2, k, k, r1, std=(k * k * r1) ** -0.5)
        self.A = self.B = None
        if self.train:
            self.A, self.B = m.empty(N, hw, hw, r1), m.empty(N, ho, wo, r2)
            self.dY, self.dX = m.normal(N, ho, wo, S), m.empty(N, hw, hw, C)
            self.dP1 = None if self.mask & 1 else m.empty(r1, C, dt=F32)
            self.dG = None if self.mask & 2 else m.empty(r2, k, k, r1, dt=F32)
            self.dP2 = None if self.mask & 4 else m.empty(S, r2, dt=F32)
        self.ws = _workspace(lrd.tucker_conv_workspace_bytes(self.g, lrd.BF16, self.mask))

    def run(self):
        lrd.tucker_conv_fwd(self.X, self.P1, self.G, self.P2, self.Y, self.A, self.B, self.g, self.ws)
        if not self.train:
            return self.Y
        lrd.tucker_conv_bwd(self.dY, self.X, self.A, self.B, self.P1, self.G, self.P2, self.dX, self.dP1, self.dG, self.dP2, self.mask, self.g,
                            self.ws)
        return dict(Y=self.Y, A=self.A, B=self.B, dX=self.dX, dP1=self.dP1, dG=self.dG, dP2=self.dP2)


_STATES = dict(layer=_Layer, stack=_Stack, encoder=_Encoder, conv=_Conv)


def prepare(case, seed):
    return _STATES[case["path"]](case, seed)


def run(state):
    return state.run()


# ------------------------------------------------------------------------------ what a pass cannot do without
def _pair_work(T, n_in, n_out, r, mask, e=2, train=True, want_h=True):
    """Activations and factors read once, results written once; H is stored and read again only where dU needs it."""
    tv, tu = train and not mask & 1, train and not mask & 2
    flops = 2 * T * r * (n_in + n_out) * (2 if train else 1) + (2 * T * r * n_out if tu else 0) + (2 * T * r * n_in if tv else 0)
    nbytes = e * (T * (n_in + n_out) + r * (n_in + n_out))
    if train:
        nbytes += e * (T * (n_in + n_out) + r * (n_in + n_out))
        nbytes += (e * T * n_in + 4 * r * n_in) * tv + (2 * e * T * r + 4 * r * n_out) * tu
    return nbytes, flops


def work(case):
    c = case
    if c["path"] == "layer":
        train = c["direction"] == "train"
        nbytes, flops = _pair_work(c["tokens"], c["n_in"], c["n_out"], c["rank"], c["mask"], 4 if c["dtype"] == "f32" else 2, train)
        if c["update"]:     # masters and momenta read and written, the compute copy written, no gradient stored
            n = c["rank"] * (c["n_in"] * (not c["mask"] & 1) + c["n_out"] * (not c["mask"] & 2))
            nbytes += n * (16 + 2 - 4)
        return dict(bytes=nbytes, flops=flops)
    if c["path"] == "stack":
        T, d, ff, r, L = c["tokens"], c["width"], c["ff"], c["rank"], c["layers"]
        pairs = [_pair_work(T, d, ff, r, c["mask"]), _pair_work(T, ff, d, r, c["mask"])]
        extra = 2 * (2 * T * ff)        # the activation beside the pre-activation, and the pre-activation read by its gradient
        return dict(bytes=L * (sum(b for b, _ in pairs) + extra), flops=L * sum(f for _, f in pairs))
    if c["path"] == "encoder":
        T, d, ff, r, L = c["tokens"], c["width"], c["ff"], c["rank"], c["layers"]
        pairs = [_pair_work(T, d, d, r, c["mask"])] * 4 + [_pair_work(T, d, ff, r, c["mask"]), _pair_work(T, ff, d, r, c["mask"])]
        shared = 2 * T * d * (2 + 2 + 2 * (not c["mask"] & 1))     # Q/K/V read one input and give one gradient
        return dict(bytes=L * (sum(b for b, _ in pairs) - shared + 4 * T * ff), flops=L * sum(f for _, f in pairs))
    N, hw, C, S, r1, r2 = c["images"], c["size"], c["c_in"], c["c_out"], c["r1"], c["r2"]
    ho = (hw - 1) // c["stride"] + 1
    pin, pout = N * hw * hw, N * ho * ho
    parts = (2 * pin * C * r1, 2 * pout * 9 * r1 * r2, 2 * pout * r2 * S)
    weights = 2 * (r1 * C + 9 * r1 * r2 + r2 * S)
    flops, nbytes = sum(parts), 2 * (pin * C + pout * S) + weights
    if c["direction"] == "train":
        flops, nbytes = 2 * flops, 2 * nbytes
        if not c["mask"] & 1:
            flops, nbytes = flops + parts[0], nbytes + 2 * pin * C + 4 * r1 * C
        if not c["mask"] & 2:
            flops, nbytes = flops + parts[1], nbytes + 2 * 2 * pin * r1 + 4 * 9 * r1 * r2
        if not c["mask"] & 4:
            flops, nbytes = flops + parts[2], nbytes + 2 * 2 * pout * r2 + 4 * r2 * S
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    # Against the same pass in 64 bits: 6e-7 in fp32; in bf16 1.7e-3 after one rounding, 2.3e-3 to 2.9e-3 after the two or
    # three of a layer, 4.8e-3 through an encoder layer's chain, 1.2e-2 through the twelve blocks of the FFN stack.
    if case.get("dtype") == "f32":
        return dict(rel=5e-6)
    return dict(rel={"stack": 3e-2, "encoder": 1.6e-2}.get(case["path"], 1e-2))
