"""The calls whose speed this library is judged by, and how each is checked.

Every case is one pass through the public entry points (``sb``, ``stack``)
on tensors that are already on the GPU, as a training program holds them.  ``listed()`` are fixed sizes, ``draw()`` gives more of the same
ranges.  Kinds of case:

``conv``   one 3x3 convolution layer of a training step: forward with bias
           and ReLU, data gradient behind the ReLU of the layer below, weight
           and bias gradient.  Filters come unpacked, as an optimiser leaves
           them.
``stack``  a block of convolutions with its pooling (``stack.ConvStack``):
           filter packing, forward with fused pooling, backward.
``fc``     one FC column shard, forward and backward on the gathered batch.
``group``  the model-parallel part of a training step of an MP group
           (``stack.GroupTrainStep.iteration`` for every modulo iteration):
           modulo and shard layers, FC shards, loss, FC updates.
``sync``   the SGD update of several replicas' conv parameters, then model
           averaging over the replicas.
"""
import math

import torch

from paper_2112_15317_amd import configs, sb, stack

POOL = configs.POOL
DEV = "cuda"

# Conv schedules by name; "pair" is two convs of `k` channels and a pool.
SCHEDULES = {"vgg16": configs.VGG16, "paper": configs.PAPER_VARIANT_CONV}


def listed():
    return [
        # The smallest call: the single RGB layer on eight images, where launches count.
        dict(name="conv_rgb_f32", kind="conv", dtype="f32", layout="nchw", n=8, c=3, h=32, w=32, k=64),
        # VGG-16 on 32x32 images, local batch 128: early, middle and late layers.
        dict(name="conv_32x32_f32", kind="conv", dtype="f32", layout="nchw", n=128, c=64, h=32, w=32, k=64),
        dict(name="conv_8x8_f32", kind="conv", dtype="f32", layout="nchw", n=128, c=256, h=8, w=8, k=256),
        dict(name="conv_4x4_f32", kind="conv", dtype="f32", layout="nchw", n=128, c=512, h=4, w=4, k=512),
        # Nothing a multiple of anything: a caller's own network.
        dict(name="conv_odd_f32", kind="conv", dtype="f32", layout="nchw", n=19, c=75, h=27, w=45, k=107),
        # bf16 activations in the caller's NCHW layout, ragged.
        dict(name="conv_odd_bf16", kind="conv", dtype="bf16", layout="nchw", n=24, c=100, h=30, w=22, k=72),
        # ImageNet-shaped block in channel-blocked bf16: packing, fused pooling, backward.
        dict(name="block_112x112_bf16", kind="stack", schedule="pair", dtype="bf16", layout="c8",
             n=32, c=64, hw=112, k=128),
        # One worker's shard of a 4096 -> 4096 FC layer on the batch gathered from four.
        dict(name="fc_shard_f32", kind="fc", dtype="f32", m=512, k_in=4096, ns=1024, relu=False),
        # A ragged bf16 shard with its ReLU.
        dict(name="fc_odd_bf16", kind="fc", dtype="bf16", m=200, k_in=1500, ns=700, relu=True),
        # K = 2 modulo iterations of the paper's variant: many small calls.
        dict(name="group_k2_f32", kind="group", mp=2, n=128, hidden=1024, classes=10),
        # Four replicas of VGG-16's conv parameters: update, then averaging.
        dict(name="sync_vgg16_f32", kind="sync", schedule="vgg16", replicas=4),
        # A whole conv step: VGG-16 on 32x32 images, forward and backward.
        dict(name="vgg16_step_f32", kind="stack", schedule="vgg16", dtype="f32", layout="nchw",
             n=128, c=3, hw=32, k=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["conv"] * 5 + ["c8"] * 2 + ["fc"] * 3 + ["stack", "group", "sync"])
    if kind in ("conv", "c8"):
        c8 = kind == "c8"
        while True:
            h = _log(rng, 8, 112) if c8 else _log(rng, 2, 64)
            w = h if rng.random() < 0.6 else max(8 if c8 else 2, int(h * rng.uniform(0.6, 1.6)))
            c = 3 if rng.random() < 0.12 and not c8 else _log(rng, 16, 512)
            k = c if rng.random() < 0.4 and c > 3 else _log(rng, 16, 512)
            n = _log(rng, 4, 128)
            if c8:
                c, k = -(-c // 8) * 8, -(-k // 8) * 8
            elif rng.random() < 0.5:
                c, k = (c if c == 3 else -(-c // 16) * 16), -(-k // 16) * 16
            fl = 18.0 * n * c * k * h * w
            if 1e7 < fl < (6e10 if c8 else 1.2e10) and n * max(c, k) * h * w < 4e7:
                break
        dt = "bf16" if c8 or rng.random() < 0.2 else "f32"
        return dict(kind="conv", dtype=dt, layout="c8" if c8 else "nchw", n=n, c=c, h=h, w=w, k=k)
    if kind == "fc":
        while True:
            m, ki, ns = _log(rng, 32, 1024), _log(rng, 128, 8192), _log(rng, 64, 2048)
            if rng.random() < 0.5:
                m, ki, ns = -(-m // 32) * 32, -(-ki // 32) * 32, -(-ns // 32) * 32
            if m * ki * ns < 2.2e9:
                break
        return dict(kind="fc", dtype=rng.choice(["f32", "f32", "bf16"]), m=m, k_in=ki, ns=ns,
                    relu=rng.random() < 0.5)
    if kind == "stack":
        if rng.random() < 0.5:
            return dict(kind="stack", schedule=rng.choice(["vgg16", "paper"]), dtype="f32",
                        layout="nchw", n=rng.randrange(9, 121), c=3, hw=32, k=0)
        hw = 2 * rng.randrange(7, 50)
        return dict(kind="stack", schedule="pair", dtype="bf16", layout="c8",
                    n=max(2, min(64, int(3e5 / (hw * hw)))), c=8 * rng.randrange(4, 24), hw=hw,
                    k=8 * rng.randrange(4, 24))
    if kind == "group":
        mp = rng.choice([1, 2, 4])
        return dict(kind="group", mp=mp, n=mp * rng.randrange(8, 128 // mp + 1),
                    hidden=mp * 4 * rng.randrange(16, 256 // mp + 1), classes=mp * rng.randrange(3, 60))
    return dict(kind="sync", schedule=rng.choice(["vgg16", "paper"]), replicas=rng.randrange(2, 7))


# ---------------------------------------------------------------- inputs --
class _Draw:
    """Seeded tensors on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed) * 7919 + 17)

    def normal(self, *shape, std=1.0):
        return torch.randn(*shape, generator=self.g, device=DEV) * std

    def act(self, *shape):
        """A ReLU output."""
        return torch.relu(self.normal(*shape))

    def grad(self, *shape):
        """An output gradient: zero-mean, small, as behind a batch mean."""
        return self.normal(*shape, std=1e-2)

    def conv_w(self, k, c):
        return self.normal(k, c, 3, 3, std=math.sqrt(2.0 / (9.0 * c)))

    def xavier(self, i, o):
        a = math.sqrt(6.0 / (i + o))
        return (torch.rand(i, o, generator=self.g, device=DEV) * 2 - 1) * a


def _to_c8(t):
    n, c, h, w = t.shape
    return t.reshape(n, c // 8, 8, h, w).permute(0, 1, 3, 4, 2).contiguous()


def _from_c8(t):
    n, cb, h, w, e = t.shape
    return t.permute(0, 1, 4, 2, 3).reshape(n, cb * e, h, w)


def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _conv_inputs(case, seed):
    """NCHW tensors in the storage type."""
    d = _Draw(seed)
    n, c, h, w, k = (case[i] for i in "nchwk")
    dt = _torch_dtype(case)
    x = d.normal(n, c, h, w) if c == 3 else d.act(n, c, h, w)
    return dict(x=x.to(dt), w=d.conv_w(k, c).to(dt), b=d.normal(k, std=0.05),
                dy=d.grad(n, k, h, w).to(dt))


def _fc_inputs(case, seed):
    d = _Draw(seed)
    m, ki, ns = case["m"], case["k_in"], case["ns"]
    dt = _torch_dtype(case)
    return dict(x=d.act(m, ki).to(dt), w=d.xavier(ki, ns).to(dt), b=d.normal(ns, std=0.05),
                dy=d.grad(m, ns).to(dt), mask=d.act(m, ns).to(dt) if case["relu"] else None)


def _schedule(case):
    if case["schedule"] == "pair":
        return [case["k"], case["k"], POOL]
    return SCHEDULES[case["schedule"]]


def _stack_inputs(case, seed):
    d = _Draw(seed)
    layers = configs.conv_layers(_schedule(case), case["c"], case["hw"])
    last = layers[-1]
    x = (d.normal if case["c"] == 3 else d.act)(case["n"], case["c"], case["hw"], case["hw"])
    return dict(layers=layers, x=x, w=[d.conv_w(l.k, l.c) for l in layers],
                b=[d.normal(l.k, std=0.05) for l in layers],
                dy=d.grad(case["n"], last.k, last.h // 2, last.w // 2))


def _group_layers(case):
    h = case["hidden"]
    return [(4096, h), (h, h), (h, case["classes"])]


def _group_inputs(case, seed):
    d = _Draw(seed)
    K, B = case["mp"], case["n"]
    fc = _group_layers(case)
    return dict(local=d.act(K, B, 4096), w=[d.xavier(i, o) for i, o in fc],
                b=[d.normal(o, std=0.02) for _, o in fc],
                labels=torch.randint(0, case["classes"], (K, B), generator=d.g, device=DEV,
                                     dtype=torch.int32))


def _sync_inputs(case, seed):
    d = _Draw(seed)
    shapes = []
    for l in configs.conv_layers(SCHEDULES[case["schedule"]], 3, 32):
        shapes += [(l.k, l.c, 3, 3), (l.k,)]
    R = case["replicas"]
    return dict(w=[[d.normal(*s, std=0.05) for s in shapes] for _ in range(R)],
                g=[[d.normal(*s, std=1e-2) for s in shapes] for _ in range(R)])


# --------------------------------------------------------------- prepare --
def _ws(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    return {"conv": _prepare_conv, "stack": _prepare_stack, "fc": _prepare_fc,
            "group": _prepare_group, "sync": _prepare_sync}[case["kind"]](case, seed)


def _prepare_conv(case, seed):
    t = _conv_inputs(case, seed)
    n, c, h, w, k = (case[i] for i in "nchwk")
    code = sb.SB_BF16 if case["dtype"] == "bf16" else sb.SB_F32
    c8 = case["layout"] == "c8"
    lay = sb.SB_NCHW8C if c8 else sb.SB_NCHW
    df = sb.conv_desc(n, c, h, w, k, code, relu=True, layout=lay)
    db = sb.conv_desc(n, c, h, w, k, code, layout=lay)
    need = max(sb.sb_conv3x3_workspace_bytes(df, sb.SB_PASS_FWD),
               sb.sb_conv3x3_workspace_bytes(db, sb.SB_PASS_BWD_DATA),
               sb.sb_conv3x3_workspace_bytes(db, sb.SB_PASS_BWD_WEIGHT))
    put = _to_c8 if c8 else (lambda a: a)
    x, dy = put(t["x"]), put(t["dy"])
    return dict(kind="conv", df=df, db=db, x=x, w=t["w"], b=t["b"], dy=dy, ws=_ws(need),
                y=torch.empty_like(dy), dx=torch.empty_like(x),
                dw=torch.empty(k, c, 3, 3, device=DEV), dbias=torch.empty(k, device=DEV),
                mask=x if c != 3 else None)


def _prepare_stack(case, seed):
    t = _stack_inputs(case, seed)
    st = stack.ConvStack(_schedule(case), case["n"], case["c"], case["hw"], case["dtype"], DEV,
                         layout=case["layout"])
    put = _to_c8 if case["layout"] == "c8" else (lambda a: a)
    dt = _torch_dtype(case)
    st.A[0].copy_(put(t["x"].to(dt)))
    for i in range(len(t["w"])):
        st.W[i].copy_(t["w"][i])
        st.b[i].copy_(t["b"][i])
    st.gA[-1].copy_(put(t["dy"].to(dt)))
    return dict(kind="stack", st=st)


def _prepare_fc(case, seed):
    t = _fc_inputs(case, seed)
    m, ki, ns = case["m"], case["k_in"], case["ns"]
    code = sb.SB_BF16 if case["dtype"] == "bf16" else sb.SB_F32
    df = sb.fc_desc(m, ki, ns, code, relu=case["relu"])
    db = sb.fc_desc(m, ki, ns, code)
    ws = _ws(max(sb.sb_fc_workspace_bytes(df, sb.SB_FC_FWD), sb.sb_fc_workspace_bytes(db, sb.SB_FC_BWD)))
    return dict(t, kind="fc", df=df, db=db, ws=ws, y=torch.empty_like(t["dy"]),
                dx=torch.empty_like(t["x"]), dw=torch.empty(ki, ns, device=DEV),
                dbias=torch.empty(ns, device=DEV))


def _plan(case):
    K = case["mp"]
    h = case["hidden"]
    lin = [("linear", i, o // K, o, j < 2) for j, (i, o) in enumerate(_group_layers(case))]
    plan = [("modulo", 4096)]
    for e in lin:
        plan += [e, ("shard", e[2], e[3])]
    return plan + [("loss", case["classes"])]


def _prepare_group(case, seed):
    t = _group_inputs(case, seed)
    K = case["mp"]
    gs = stack.GroupTrainStep(configs.PAPER_VARIANT_CONV, case["n"], 3, 32, _plan(case), device=DEV)
    gs.local.copy_(t["local"])
    for j, (i, o) in enumerate(_group_layers(case)):
        gs.W[j].copy_(t["w"][j].reshape(i, K, o // K).permute(1, 0, 2))
        gs.b[j].copy_(t["b"][j].reshape(K, o // K))
    gs.labels.copy_(t["labels"])
    return dict(kind="group", gs=gs)


def _prepare_sync(case, seed):
    t = _sync_inputs(case, seed)
    lists = [sb.SgdList([(w, g, 1.0) for w, g in zip(ws, gs)]) for ws, gs in zip(t["w"], t["g"])]
    return dict(kind="sync", t=t, lists=lists, sets=[list(s) for s in zip(*t["w"])])


# ------------------------------------------------------------------- run --
def run(s):
    kind = s["kind"]
    if kind == "conv":
        sb.sb_conv3x3_fwd(s["df"], s["x"], s["w"], s["b"], s["y"], s["ws"])
        sb.sb_conv3x3_bwd_data(s["db"], s["dy"], s["w"], s["mask"], s["dx"], s["ws"])
        sb.sb_conv3x3_bwd_weight(s["db"], s["x"], s["dy"], s["dw"], s["dbias"], s["ws"])
        return dict(y=s["y"], dx=s["dx"], dw=s["dw"], db=s["dbias"])
    if kind == "stack":
        st = s["st"]
        st.step()
        return dict(y=st.A[-1], dx=st.gA[0], dw=st.dW, db=st.db)
    if kind == "fc":
        sb.sb_fc_shard_fwd(s["df"], s["x"], s["w"], s["b"], s["y"], s["ws"])
        sb.sb_fc_shard_bwd(s["db"], s["x"], s["w"], s["dy"], s["mask"], s["dx"], s["dw"], s["dbias"],
                           False, s["ws"])
        return dict(y=s["y"], dx=s["dx"], dw=s["dw"], db=s["dbias"])
    if kind == "group":
        gs = s["gs"]
        for k in range(gs.K):
            gs.iteration(k)
        return dict(logits=gs.X[-1], loss=gs.loss, dlocal=gs.dlocal, w=gs.W, b=gs.b)
    for sl in s["lists"]:
        sb.sb_sgd_update(sl, 0.01)
    for ts in s["sets"]:
        sb.sb_model_average_replicas(ts)
    return dict(w=s["t"]["w"][0])


# ------------------------------------------------------------------ work --
def _valid(n):
    """In-image (position, tap) pairs of a 3-tap axis with padding 1."""
    return 3 * n - 2 if n > 1 else 1


def _conv_work(n, c, h, w, k, es, passes=3):
    act = n * h * w * es
    flops = 2.0 * n * c * k * _valid(h) * _valid(w) * passes
    # Forward: x, w, b -> y.  Data gradient: dy, w, mask -> dx.  Weight gradient: x, dy -> dw, db.
    by = act * (c + k) + act * (k + 2 * c) + act * (c + k) + 2.0 * k * c * 9 * es + k * c * 9 * 4 + 8 * k
    return by, flops


def work(case):
    kind = case["kind"]
    es = 2 if case.get("dtype") == "bf16" else 4
    if kind == "conv":
        by, fl = _conv_work(*(case[i] for i in "nchwk"), es)
    elif kind == "stack":
        by = fl = 0.0
        for l in configs.conv_layers(_schedule(case), case["c"], case["hw"]):
            a, f = _conv_work(case["n"], l.c, l.h, l.w, l.k, es)
            by, fl = by + a, fl + f
            if l.pool_after:   # codes written and read, the gradient spread over the windows
                by += case["n"] * l.k * l.h * l.w * (es + 0.5)
    elif kind == "fc":
        m, ki, ns = case["m"], case["k_in"], case["ns"]
        fl = 6.0 * m * ki * ns
        by = es * (3.0 * m * ki + 2.0 * ki * ns + (4 if case["relu"] else 3) * m * ns) + 4.0 * ki * ns
    elif kind == "group":
        K, B = case["mp"], case["n"]
        fl = by = 0.0
        for i, o in _group_layers(case):
            fl += 6.0 * B * i * o
            by += 4.0 * (6.0 * i * o + 3.0 * B * (i + o) + K * B * i)
        by, fl = by * K, fl * K
    else:
        p = sum(l.k * l.c * 9 + l.k for l in configs.conv_layers(SCHEDULES[case["schedule"]], 3, 32))
        R = case["replicas"]
        by, fl = 4.0 * p * R * 5, 4.0 * p * R
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """About four times the error against 64 bits that the calls show (fp32
    sums up to 6e-7, bf16 results 1.7e-3)."""
    kind = case["kind"]
    if kind in ("conv", "fc"):
        if case["dtype"] == "bf16":
            return {"rel": 7e-3, "max": 2e-2}
        return {"rel": 3e-6, "max": 5e-5}
    if kind == "stack":
        # A changed rounding may move a pooling decision, which moves a whole gradient.
        return {"rel": 2e-2, "max": 1.0 - 1e-9}
    if kind == "group":
        # A pre-activation within rounding of zero may change sides of its
        # ReLU: one of 1e5 gradient elements then appears or vanishes.
        return {"rel": 1e-2, "max": 0.5}
    return {"rel": 3e-7, "max": 2e-6}


# ----------------------------------------------------------------- exact --
def _shift(xp, r, s, h, w):
    """Channel-major [c, n*h*w] window (r, s) of a padded [c, n, h+2, w+2] tensor."""
    return xp[:, :, r:r + h, s:s + w].reshape(xp.shape[0], -1)


def _conv_fwd64(x, w, b):
    n, c, h, wd = x.shape
    xp = torch.nn.functional.pad(x.permute(1, 0, 2, 3).contiguous(), (1, 1, 1, 1))
    y = torch.zeros(w.shape[0], n * h * wd, dtype=torch.float64, device=x.device)
    for r in range(3):
        for s in range(3):
            y += w[:, :, r, s].contiguous() @ _shift(xp, r, s, h, wd)
    if b is not None:
        y += b[:, None]
    return y.reshape(-1, n, h, wd).permute(1, 0, 2, 3)


def _conv_bwd64(x, w, dy):
    n, c, h, wd = x.shape
    dx = _conv_fwd64(dy, w.flip(2, 3).transpose(0, 1).contiguous(), None)
    xp = torch.nn.functional.pad(x.permute(1, 0, 2, 3).contiguous(), (1, 1, 1, 1))
    g = dy.permute(1, 0, 2, 3).reshape(dy.shape[1], -1)
    dw = torch.stack([torch.stack([g @ _shift(xp, r, s, h, wd).t().contiguous() for s in range(3)], -1)
                      for r in range(3)], -2)
    return dx, dw, g.sum(1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "conv":
        t = _conv_inputs(case, seed)
        x, w, b, dy = (t[i].double() for i in ("x", "w", "b", "dy"))
        y = torch.relu(_conv_fwd64(x, w, b))
        dx, dw, db = _conv_bwd64(x, w, dy)
        if case["c"] != 3:
            dx = dx * (x > 0)
        if case["layout"] == "c8":
            y, dx = _to_c8(y), _to_c8(dx)
        return dict(y=y.contiguous(), dx=dx.contiguous(), dw=dw.contiguous(), db=db)
    if kind == "stack":
        # The forward alone: near-ties of the pooling make the gradient's exact value arbitrary.
        t = _stack_inputs(case, seed)
        dt = _torch_dtype(case)
        a = t["x"].to(dt).double()
        for i, l in enumerate(t["layers"]):
            a = torch.relu(_conv_fwd64(a, t["w"][i].to(dt).double(), t["b"][i].double()))
            if l.pool_after:
                a = a.reshape(a.shape[0], a.shape[1], l.h // 2, 2, l.w // 2, 2).amax((3, 5))
        if case["layout"] == "c8":
            a = _to_c8(a)
        none = [None] * len(t["w"])
        return dict(y=a.contiguous(), dx=None, dw=none, db=none)
    if kind == "fc":
        t = {k: v.double() if v is not None else None for k, v in _fc_inputs(case, seed).items()}
        y = t["x"] @ t["w"] + t["b"]
        g = t["dy"] if t["mask"] is None else t["dy"] * (t["mask"] > 0)
        return dict(y=torch.relu(y) if case["relu"] else y, dx=g @ t["w"].t().contiguous(),
                    dw=t["x"].t().contiguous() @ g, db=g.sum(0))
    if kind == "group":
        return _exact_group(case, seed)
    t = _sync_inputs(case, seed)
    lr = float(torch.tensor(0.01, dtype=torch.float32))
    out = []
    for i in range(len(t["w"][0])):
        out.append(sum(w[i].double() - lr * g[i].double() for w, g in zip(t["w"], t["g"]))
                   / case["replicas"])
    return dict(w=out)


def _exact_group(case, seed):
    t = _group_inputs(case, seed)
    K, B = case["mp"], case["n"]
    s = B // K
    local = t["local"].double()
    w, b = [v.double() for v in t["w"]], [v.double() for v in t["b"]]
    lr = float(torch.tensor(0.01, dtype=torch.float32)) / K
    dlocal = torch.zeros_like(local)
    losses = []
    for k in range(K):
        rows = slice(k * s, k * s + s)
        a = [local[:, rows].reshape(B, -1)]
        for j in range(3):
            z = a[j] @ w[j] + b[j]
            a.append(torch.relu(z) if j < 2 else z)
        logp = torch.log_softmax(a[3], 1)
        lab = t["labels"][k].long()
        losses.append(-logp.gather(1, lab[:, None])[:, 0])
        g = logp.exp()
        g[torch.arange(B, device=DEV), lab] -= 1.0
        g = g / B
        for j in reversed(range(3)):
            if j < 2:
                g = g * (a[j + 1] > 0)
            dw, db = a[j].t().contiguous() @ g, g.sum(0)
            g = g @ w[j].t().contiguous()
            w[j], b[j] = w[j] - lr * dw, b[j] - lr * db
        dlocal[:, rows] = g.reshape(K, s, -1)
        logits = a[3]
    shard = lambda v: v.reshape(v.shape[0], K, -1).permute(1, 0, 2).contiguous()
    return dict(logits=logits, loss=torch.stack(losses), dlocal=dlocal, w=[shard(v) for v in w],
                b=[v.reshape(K, -1) for v in b])
