"""The workloads whose speed this framework is judged by, through its public
entry points: whole forward passes and training steps of the convolution
stack (``ConvStack``), single layers of it with their backward, the unfused
elementwise and pooling passes, the fully-connected head (``FCHead``) and the
parameter update (``cf_adam_larc_step``).

A case is a dict of plain values; ``kind`` says which of these it is:

  infer    forward of a ConvStack of ``depth`` layers, ``size``^3 x ``c0``
           cubes, ``batch`` of them, ``dtype``
  step     the same network forward and backward: output and all gradients
  layer    one layer (``cin``, ``cout``, ``k``, ``stride``, ``pad``, ``pool``)
           forward and backward: output, dW, db and, from 16 input channels
           on, dx
  passes   bias + leaky ReLU and 2^3 average pool, forward and backward, as
           the separate unfused calls
  head     the three-layer head: forward, loss and backward
  update   one Adam + LARC step over ``groups`` tensors of ``params`` values

``exact`` evaluates the same definitions in float64 with torch alone.
"""
import math

import torch

from paper_1808_04728_amd import binding as B
from paper_1808_04728_amd import inputs
from paper_1808_04728_amd.head import FCHead
from paper_1808_04728_amd.stack import ConvStack

ALPHA = inputs.ALPHA
DEV = "cuda:0"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest call: the first layer alone on one small cube, where the
        # launch and the host's share of a call are what a user waits for
        dict(name="infer_layer1_32_f32", kind="infer", depth=1, c0=1, c5=128, size=32, batch=1, dtype="f32"),
        # prediction from a trained network: forward only, bf16, one cube whose
        # side is no power of two (100 -> 50 -> 25 -> 13 -> 6)
        dict(name="infer_100_bf16_b1", kind="infer", depth=6, c0=1, c5=128, size=100, batch=1, dtype="bf16"),
        # a training step on small cubes: every kernel takes a few microseconds
        dict(name="step_64_f32_b1", kind="step", depth=6, c0=1, c5=128, size=64, batch=1, dtype="f32"),
        # the paper's workload: one 128^3 cube per device in fp32
        dict(name="step_128_f32_b1", kind="step", depth=6, c0=1, c5=128, size=128, batch=1, dtype="f32"),
        # the throughput workload: eight 128^3 cubes in bf16
        dict(name="step_128_bf16_b8", kind="step", depth=6, c0=1, c5=128, size=128, batch=8, dtype="bf16"),
        # the first layer of the scaled-up network: four input fields of 256^3
        dict(name="layer1_c4_256_bf16_b2", kind="layer", cin=4, cout=16, k=3, stride=1, pad="same", pool=True, size=256,
             batch=2, dtype="bf16"),
        # the paper's second layer in fp32 on cubes of an odd side
        dict(name="layer2_45_f32_b2", kind="layer", cin=16, cout=32, k=4, stride=1, pad="same", pool=True, size=45, batch=2,
             dtype="f32"),
        # the paper's third layer (VALID, stride 1), where its network has most channels times voxels
        dict(name="layer3_valid_30_bf16_b8", kind="layer", cin=32, cout=64, k=4, stride=1, pad="valid", pool=True, size=30,
             batch=8, dtype="bf16"),
        # a deep layer on an odd side: little work per voxel row, many channels
        dict(name="layer4_13_bf16_b4", kind="layer", cin=64, cout=64, k=3, stride=1, pad="same", pool=False, size=13,
             batch=4, dtype="bf16"),
        # a program that calls the unfused activation and pooling passes, at the
        # first layer's activation
        dict(name="passes_128_bf16_b8", kind="passes", c=16, size=128, batch=8, dtype="bf16"),
        # the head of the eight-cube step
        dict(name="head_65536_bf16_b8", kind="head", features=65536, batch=8, dtype="bf16"),
        # the update of a network of the paper's parameter count (7.04 M)
        dict(name="update_7m_f32", kind="update", params=7037500, groups=20, dtype="f32"),
    ]


#: the network's layers past the first, with the sides at which it meets them
_LAYERS = [
    dict(cin=16, cout=32, k=4, stride=1, pad="same", pool=True, lo=16, hi=64),
    dict(cin=16, cout=32, k=4, stride=1, pad="valid", pool=True, lo=16, hi=64),
    dict(cin=32, cout=64, k=4, stride=2, pad="same", pool=True, lo=12, hi=64),
    dict(cin=32, cout=64, k=4, stride=1, pad="valid", pool=True, lo=12, hi=32),
    dict(cin=64, cout=64, k=3, stride=1, pad="same", pool=False, lo=4, hi=16),
    dict(cin=64, cout=128, k=2, stride=1, pad="same", pool=False, lo=4, hi=16),
    dict(cin=128, cout=128, k=2, stride=1, pad="same", pool=False, lo=4, hi=16),
    dict(cin=256, cout=256, k=2, stride=1, pad="same", pool=False, lo=4, hi=16),
]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges the listed ones stand for: any side, not
    only powers of two, batches from 1 to 8, both types.  Work is held below
    the largest listed cases' (about 64 GFLOP in fp32, 480 in bf16, 34 M
    input voxels)."""
    while True:
        kind = rng.choice(["infer", "step", "step", "layer", "layer", "layer", "passes", "head", "update"])
        dtype = rng.choice(["f32", "bf16"])
        batch = rng.choice([1, 1, 2, 3, 4, 8])
        if kind in ("infer", "step"):
            c = dict(kind=kind, depth=rng.choice([1, 6]) if kind == "infer" else 6, c0=rng.choice([1, 1, 1, 4]), c5=128,
                     size=_log(rng, 32, 144), batch=batch, dtype=dtype)
        elif kind == "layer":
            if rng.random() < 0.34:
                c = dict(kind=kind, cin=rng.choice([1, 1, 4]), cout=16, k=3, stride=1, pad=rng.choice(["same", "valid"]),
                         pool=True, size=_log(rng, 24, 256), batch=batch, dtype=dtype)
            else:
                spec = dict(rng.choice(_LAYERS))
                lo, hi = spec.pop("lo"), spec.pop("hi")
                c = dict(kind=kind, **spec, size=_log(rng, lo, hi), batch=batch, dtype=dtype)
        elif kind == "passes":
            c = dict(kind=kind, c=rng.choice([16, 32, 64]), size=_log(rng, 8, 128), batch=batch, dtype=dtype)
        elif kind == "head":
            c = dict(kind=kind, features=128 * _log(rng, 8, 512), batch=rng.randint(1, 8), dtype=dtype)
        else:
            c = dict(kind=kind, params=_log(rng, 400000, 16000000), groups=rng.randint(8, 24), dtype=dtype)
        w = work(c)
        if w["flops"] <= (64e9 if dtype == "f32" else 480e9) and w["bytes"] <= 3.9e9 and not (
                kind in ("infer", "step", "layer") and c["batch"] * c["size"] ** 3 > 2 * 256 ** 3):
            return c


# ---------------------------------------------------------------------------
# shapes and work
# ---------------------------------------------------------------------------

def _out(n, k, s, pad):
    """(output extent, padding before) of one dimension."""
    if pad == "same":
        o = -(-n // s)
        return o, max((o - 1) * s + k - n, 0) // 2
    return (n - k) // s + 1, 0


def _layers(case):
    """[(layer spec, input side, output side, side after the pool)]"""
    if case["kind"] == "layer":
        specs = [{n: case[n] for n in ("cin", "cout", "k", "stride", "pad", "pool")}]
    else:
        specs = inputs.stack_layers(case["c0"], case["c5"])[:case["depth"]]
    r, n = [], case["size"]
    for s in specs:
        o, _ = _out(n, s["k"], s["stride"], s.get("pad", "same"))
        p = o // 2 if s["pool"] else o
        r.append((s, n, o, p))
        n = p
    return r


def _es(case):
    return 2 if case["dtype"] == "bf16" else 4


def _needs_dx(case):
    return case["kind"] == "layer" and case["cin"] >= 16


def work(case):
    """Bytes: every input read once, every output written once (of each call,
    where the pass is several calls).  FLOPs: two per product of a tap inside
    the input."""
    es, kind = _es(case), case["kind"]
    if kind in ("infer", "step", "layer"):
        L, b = _layers(case), case["batch"]
        flops = params = 0
        for i, (s, n, o, p) in enumerate(L):
            _, before = _out(n, s["k"], s["stride"], s.get("pad", "same"))
            taps = sum(min(n, a * s["stride"] - before + s["k"]) - max(0, a * s["stride"] - before) for a in range(o))
            f = 2 * b * taps ** 3 * s["cin"] * s["cout"]
            flops += f * (1 if kind == "infer" else 3 if i > 0 or _needs_dx(case) else 2)
            params += s["k"] ** 3 * s["cin"] * s["cout"] + s["cout"]
        first, last = L[0], L[-1]
        xb = b * first[1] ** 3 * first[0]["cin"] * es
        yb = b * last[3] ** 3 * last[0]["cout"] * es
        nbytes = xb + yb + params * es
        if kind != "infer":
            nbytes += yb + params * 4 + (xb if _needs_dx(case) else 0)
        return dict(bytes=nbytes, flops=flops)
    if kind == "passes":
        z = case["batch"] * case["size"] ** 3 * case["c"]
        p = case["batch"] * (case["size"] // 2) ** 3 * case["c"]
        # four separate calls: z -> y, y -> p, dp -> dy, (dy, y) -> dz
        return dict(bytes=(7 * z + 2 * p) * es, flops=8 * z)
    if kind == "head":
        dims, m = [case["features"], *inputs.HEAD_WIDTHS], case["batch"]
        w = sum(dims[i] * dims[i + 1] for i in range(3))
        return dict(bytes=w * (es + 4) + 2 * m * dims[0] * es, flops=6 * m * w)
    n = case["params"]
    return dict(bytes=n * (28 + (2 if case["dtype"] == "bf16" else 0)), flops=16 * n)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _tdt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _cubes(batch, size, c0, g):
    """Log counts of a Poisson-sampled lognormal field with a P(k) ~ k^-2.5
    spectrum, mean 8 particles a voxel (the recipe of inputs.py, drawn on the
    GPU)."""
    f = torch.fft.fftfreq(size, device=DEV) * size
    h = torch.fft.rfftfreq(size, device=DEV) * size
    k2 = f[:, None, None] ** 2 + f[None, :, None] ** 2 + h[None, None, :] ** 2
    amp = torch.where(k2 > 0, k2.clamp_min(1.0) ** -0.625, torch.zeros_like(k2))
    x = torch.empty((batch, size, size, size, c0), device=DEV)
    s2 = math.log(3.0)
    for b in range(batch):
        for c in range(c0):
            n = torch.randn((size, size, size), generator=g, device=DEV)
            d = torch.fft.irfftn(torch.fft.rfftn(n) * amp, s=(size, size, size), dim=(0, 1, 2))
            d = (d - d.mean()) / d.std()
            rho = torch.exp(math.sqrt(s2) * d - s2 / 2)
            x[b, ..., c] = torch.log1p(torch.poisson(8.0 * rho, generator=g))
    return x


def _activations(shape, g):
    """What a layer inside the network reads: leaky ReLU of N(0, 1), averaged
    over the eight voxels of a pooling window."""
    a = torch.zeros(shape, device=DEV)
    for _ in range(8):
        u = torch.randn(shape, generator=g, device=DEV)
        a += torch.where(u > 0, u, ALPHA * u)
    return a / 8


def _conv_data(case, seed):
    """(x, weights, biases, upstream gradient or None) of a convolution case,
    in the case's type (biases fp32)."""
    g, t = _gen(seed), _tdt(case)
    L, b = _layers(case), case["batch"]
    cin = L[0][0]["cin"]
    n = case["size"]
    x = (_cubes(b, n, cin, g) if cin <= 4 else _activations((b, n, n, n, cin), g)).to(t)
    ws, bs = [], []
    for s, _, _, _ in L:
        k = s["k"]
        w = torch.randn((k, k, k, s["cin"], s["cout"]), generator=g, device=DEV) * math.sqrt(2.0 / (k ** 3 * s["cin"]))
        ws.append(w.to(t))
        bs.append(0.05 * torch.randn((s["cout"],), generator=g, device=DEV))
    dout = None
    if case["kind"] != "infer":
        p = L[-1][3]
        dout = torch.randn((b, p, p, p, L[-1][0]["cout"]), generator=g, device=DEV).to(t)
    return x, ws, bs, dout


def _passes_data(case, seed):
    g, t = _gen(seed), _tdt(case)
    b, n, c = case["batch"], case["size"], case["c"]
    z = torch.randn((b, n, n, n, c), generator=g, device=DEV).to(t)
    dp = torch.randn((b, n // 2, n // 2, n // 2, c), generator=g, device=DEV).to(t)
    bias = 0.05 * torch.randn((c,), generator=g, device=DEV)
    return z, dp, bias


def _head_data(case, seed):
    g, t = _gen(seed), _tdt(case)
    m, dims = case["batch"], [case["features"], *inputs.HEAD_WIDTHS]
    u = torch.randn((m, dims[0]), generator=g, device=DEV)
    x = torch.where(u > 0, u, ALPHA * u).to(t)
    ws = [(torch.randn((dims[i], dims[i + 1]), generator=g, device=DEV) * math.sqrt(2.0 / dims[i])).to(t) for i in range(3)]
    # early in training: the outputs are still off by more than their targets, so
    # that the loss gradient is no difference of nearly equal bf16 values
    bs = [0.05 * torch.randn((dims[i + 1],), generator=g, device=DEV) + (3.0 if i == 2 else 0.0) for i in range(3)]
    lo = torch.tensor([r[0] for r in inputs.PARAM_RANGES], device=DEV)
    hi = torch.tensor([r[1] for r in inputs.PARAM_RANGES], device=DEV)
    target = lo + (hi - lo) * torch.rand((m, 3), generator=g, device=DEV)
    return x, ws, bs, target


def _update_data(case, seed):
    """A step in the middle of training: moments that have settled around the
    rescaled gradient, weights of different scale per tensor."""
    g = _gen(seed)
    k = case["groups"]
    share = [0.2 + 0.8 * (((i * 7 + 3) * 2654435761 % 1000) / 1000) for i in range(k)]
    off = [0]
    for f in share:
        off.append(off[-1] + max(4, int(case["params"] * f / sum(share)) // 4 * 4))
    n = off[-1]
    v = torch.randn(n, generator=g, device=DEV)
    for i in range(k):
        v[off[i]:off[i + 1]] *= 0.02 * (1 + i % 5)
    gr = torch.randn(n, generator=g, device=DEV)
    m = 1e-5 * torch.randn(n, generator=g, device=DEV)
    s = 1e-10 * torch.rand(n, generator=g, device=DEV)
    return off, v, gr, m, s


UPDATE_T = 1000
T_DECAY = 100000


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------

def prepare(case, seed):
    kind, dt = case["kind"], case["dtype"]
    if kind in ("infer", "step", "layer"):
        x, ws, bs, dout = _conv_data(case, seed)
        st = ConvStack([s for s, _, _, _ in _layers(case)], case["size"], case["batch"], dt, ALPHA, DEV,
                       skip_first_dgrad=not _needs_dx(case))
        st.set_params(ws, bs)
        st.set_input(x)
        return dict(kind=kind, stack=st, dout=dout, dx=_needs_dx(case))
    if kind == "passes":
        z, dp, bias = _passes_data(case, seed)
        c = case["c"]
        nvox = z.numel() // c
        ws = torch.empty(max(16, B.cf_bias_lrelu_bwd_workspace_size(nvox, c)), dtype=torch.uint8, device=DEV)
        return dict(kind=kind, dtype=dt, z=z, dp=dp, bias=bias, nvox=nvox, c=c, shape=tuple(z.shape[:4]), y=torch.empty_like(z),
                    p=torch.empty_like(dp), dy=torch.empty_like(z), dz=torch.empty_like(z), db=torch.empty(c, device=DEV),
                    ws=ws)
    if kind == "head":
        x, ws, bs, target = _head_data(case, seed)
        head = FCHead(case["batch"], case["features"], inputs.HEAD_WIDTHS, dt, ALPHA, DEV)
        head.set_params(ws, bs, target)
        return dict(kind=kind, head=head, x=x)
    off, v, g, m, s = _update_data(case, seed)
    return dict(kind=kind, t=UPDATE_T, hp=B.make_hparams(T_DECAY), off=B.adam_offsets(off), v=v, g=g, m=m, s=s,
                v16=torch.empty(off[-1], dtype=torch.bfloat16, device=DEV) if dt == "bf16" else None,
                ws=torch.empty(max(16, B.cf_adam_larc_workspace_size(off)), dtype=torch.uint8, device=DEV))


def run(state):
    kind = state["kind"]
    if kind == "infer":
        return state["stack"].forward()
    if kind in ("step", "layer"):
        st = state["stack"]
        out = st.forward()
        st.backward(state["dout"])
        r = dict(out=out, grad=st.flat_grad)
        if state["dx"]:
            r["dx"] = st.L[0]["dx"]
        return r
    if kind == "passes":
        q, dt, c = state, state["dtype"], state["c"]
        B.cf_bias_lrelu_fwd(q["nvox"], c, dt, q["z"], q["bias"], ALPHA, q["y"])
        B.cf_avgpool3d_fwd(*q["shape"], c, 2, 2, dt, q["y"], q["p"])
        B.cf_avgpool3d_bwd(*q["shape"], c, 2, 2, dt, q["dp"], q["dy"])
        B.cf_bias_lrelu_bwd(q["nvox"], c, dt, q["dy"], q["y"], ALPHA, q["dz"], q["db"], q["ws"])
        return dict(y=q["y"], p=q["p"], dy=q["dy"], dz=q["dz"], db=q["db"])
    if kind == "head":
        h = state["head"]
        dx = h.step(state["x"])
        return dict(y=h.y, loss=h.loss[:1], dw=h.dw, db=h.db, dx=dx)
    q = state
    B.cf_adam_larc_step(q["off"], q["t"], q["hp"], q["v"], q["g"], q["m"], q["s"], q["v16"], q["ws"])
    q["t"] += 1
    return dict(v=q["v"], m=q["m"], s=q["s"], v16=q["v16"])


# ---------------------------------------------------------------------------
# tolerances and the float64 reference
# ---------------------------------------------------------------------------

def tolerance(case):
    """About four times what the path differs from the float64 reference by,
    over the listed cases and drawn ones.  A pre-activation within rounding of
    zero may take the other slope: one such voxel moves the gradients around it
    by up to half their size, and 1e-5 of them over a tensor in fp32."""
    kind, bf = case["kind"], case["dtype"] == "bf16"
    if kind == "infer":
        return {"rel": 0.015 if bf else 2e-6}
    if kind == "step":
        return {"rel": 0.03} if bf else {"rel": 2e-4, "max": 0.5}
    if kind == "layer":
        return {"rel": 0.008 if bf else 6e-5, "max": 0.5}
    if kind == "passes":
        return {"rel": 0.008 if bf else 1e-6}
    if kind == "head":
        return {"rel": 0.015 if bf else 2e-6}
    return {"rel": 0.007 if bf else 1e-7}


def _taps(s, n, o):
    """(tap index, padding) of a layer, and a function that gives the input
    voxels under one tap as a slice of the padded input."""
    k, st = s["k"], s["stride"]
    _, before = _out(n, k, st, s.get("pad", "same"))
    after = max(0, (o - 1) * st + k - n - before)

    def window(t):
        return tuple(slice(a, a + (o - 1) * st + 1, st) for a in t)

    taps = [(a, b, c) for a in range(k) for b in range(k) for c in range(k)]
    return taps, window, before, after


def _padded(x, before, after):
    return torch.nn.functional.pad(x, (0, 0, before, after, before, after, before, after))


def _conv64(x, w, s, n, o):
    taps, win, b, a = _taps(s, n, o)
    xp = _padded(x, b, a)
    z = torch.zeros((x.shape[0] * o ** 3, s["cout"]), dtype=torch.float64, device=DEV)
    for t in taps:
        v = xp[(slice(None),) + win(t)].reshape(-1, s["cin"])
        z.addmm_(v, w[t])
    return z.view(x.shape[0], o, o, o, s["cout"])


def _conv64_grads(x, w, dz, s, n, o, need_dx):
    taps, win, b, a = _taps(s, n, o)
    xp = _padded(x, b, a)
    g = dz.reshape(-1, s["cout"])
    dw = torch.empty_like(w)
    dxp = torch.zeros_like(xp) if need_dx else None
    for t in taps:
        at = (slice(None),) + win(t)
        dw[t] = xp[at].reshape(-1, s["cin"]).t().contiguous() @ g
        if need_dx:
            dxp[at] += (g @ w[t].t().contiguous()).view(dxp[at].shape)
    return dw, dxp[:, b:b + n, b:b + n, b:b + n] if need_dx else None


def _pool64(y):
    b, n, c = y.shape[0], y.shape[1], y.shape[4]
    q = n // 2
    return y[:, :2 * q, :2 * q, :2 * q].reshape(b, q, 2, q, 2, q, 2, c).mean(dim=(2, 4, 6))


def _pool64_grad(dp, n):
    b, q, c = dp.shape[0], dp.shape[1], dp.shape[4]
    dy = torch.zeros((b, n, n, n, c), dtype=torch.float64, device=DEV)
    v = dy[:, :2 * q, :2 * q, :2 * q].view(b, q, 2, q, 2, q, 2, c) if n == 2 * q else None
    if v is not None:
        v += (dp / 8)[:, :, None, :, None, :, None, :]
    else:
        for i in range(8):
            dy[:, (i >> 2):2 * q:2, ((i >> 1) & 1):2 * q:2, (i & 1):2 * q:2] = dp / 8
    return dy


def _lrelu64(u):
    return torch.where(u > 0, u, ALPHA * u)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("infer", "step", "layer"):
        x, ws, bs, dout = _conv_data(case, seed)
        h, L, kept = x.double(), _layers(case), []
        del x
        for (s, n, o, p), w, b in zip(L, ws, bs):
            u = _conv64(h, w.double(), s, n, o) + b.double()
            kept.append((h, u > 0))
            h = _lrelu64(u)
            h = _pool64(h) if s["pool"] else h
        if kind == "infer":
            return h
        r, g, grads = dict(out=h), dout.double(), []
        for i in range(len(L) - 1, -1, -1):
            s, n, o, p = L[i]
            xin, pos = kept[i]
            dy = _pool64_grad(g, o) if s["pool"] else g
            dz = torch.where(pos, dy, ALPHA * dy)
            need = i > 0 or _needs_dx(case)
            dw, g = _conv64_grads(xin, ws[i].double(), dz, s, n, o, need)
            grads = [dw.reshape(-1), dz.sum(dim=(0, 1, 2, 3))] + grads
        # each tensor starts on a multiple of 16 values in the flat gradient, zeros between
        r["grad"] = torch.cat([torch.nn.functional.pad(t, (0, -t.numel() % 16)) for t in grads])
        if kind == "step" and case["dtype"] == "bf16":
            # six layers of bf16 activations give about 0.3% of the pre-activations
            # the other sign than 64 bits do: no bf16 gradient of the whole network
            # is nearer than 5 to 10% (the single layers' gradients are compared)
            r["grad"] = None
        if _needs_dx(case):
            r["dx"] = g
        return r
    if kind == "passes":
        z, dp, bias = _passes_data(case, seed)
        y = _lrelu64(z.double() + bias.double())
        dy = _pool64_grad(dp.double(), case["size"])
        dz = torch.where(y > 0, dy, ALPHA * dy)
        return dict(y=y, p=_pool64(y), dy=dy, dz=dz, db=dz.sum(dim=(0, 1, 2, 3)))
    if kind == "head":
        x, ws, bs, target = _head_data(case, seed)
        W, h, ys, hs = [w.double() for w in ws], x.double(), [], []
        for w, b in zip(W, bs):
            hs.append(h)
            h = _lrelu64(h @ w + b.double())
            ys.append(h)
        d = h - target.double()
        loss = (d * d).mean().reshape(1)
        g, dw, db = 2 * d / d.numel(), [None] * 3, [None] * 3
        for i in (2, 1, 0):
            dz = torch.where(ys[i] > 0, g, ALPHA * g)
            dw[i] = hs[i].t().contiguous() @ dz
            db[i] = dz.sum(dim=0)
            g = dz @ W[i].t().contiguous()
        return dict(y=ys, loss=loss, dw=dw, db=db, dx=g)
    off, v, gr, m, s = (t.double() if torch.is_tensor(t) else t for t in _update_data(case, seed))
    hp, t = B.PAPER_HPARAMS, UPDATE_T
    eta = (hp["eta0"] - hp["eta_min"]) * (1 - min(t, T_DECAY) / T_DECAY) + hp["eta_min"]
    step = eta * math.sqrt(1 - hp["beta2"] ** (t + 1)) / (1 - hp["beta1"] ** (t + 1))
    for a, b in zip(off, off[1:]):
        vn, gn = v[a:b].norm(), gr[a:b].norm()
        rate = torch.clamp(hp["larc_coef"] * vn / gn, max=hp["larc_clip"])
        q = rate * gr[a:b]
        m[a:b] = hp["beta1"] * m[a:b] + (1 - hp["beta1"]) * q
        s[a:b] = hp["beta2"] * s[a:b] + (1 - hp["beta2"]) * q * q
        v[a:b] -= step * m[a:b] / (torch.sqrt(s[a:b]) + hp["eps_hat"])
    return dict(v=v, m=m, s=s, v16=v if case["dtype"] == "bf16" else None)
