"""Workloads of the collocated stages, as a user's program runs them.

A case is one pass of one device's share of a pipeline:

* ``mode="train"``: one training iteration after a parameter update.  The
  compute copies of the weights are refreshed from the fp32 masters
  (``sync_params``), the gradients are cleared, and ``micro`` microbatches run
  forward and backward on the encoder and the decoder half; with more than one
  microbatch the schedule executor drives them.  It returns every boundary
  output, the timestep-embedding gradient and every parameter gradient.
* ``mode="sample"``: one denoising step of a trained model, the forward of
  both halves.

``kind="res"`` is the ResBlock stage (UNet levels), ``kind="tok"`` the
transformer-block stage (UViT and Hunyuan-DiT families).  ``exact`` computes
the same stage from its definition with torch in float64.
"""

import math

import torch
import torch.nn.functional as F

from paper_2606_19163_amd import configs
from paper_2606_19163_amd import stage as S
from paper_2606_19163_amd import tstage as T

_BF16, _F32 = configs.BF16, configs.F32


def _res(name, mode, dtype, batch, height, width, cin, c, groups, temb, blocks, micro, overlap):
    case = dict(kind="res", mode=mode, dtype=dtype, batch=batch, height=height, width=width,
                cin=cin, c=c, groups=groups, temb=temb, blocks=blocks, micro=micro,
                overlap=overlap)
    if name:
        case["name"] = name
    return case


def _tok(name, mode, batch, tokens, heads, mlp, blocks, micro, overlap):
    case = dict(kind="tok", mode=mode, dtype=_BF16, batch=batch, tokens=tokens, heads=heads,
                mlp=mlp, blocks=blocks, micro=micro, overlap=overlap)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # a tiny fp32 model, as first experiments and checks run it: launches count
        _res("res-f32-16x16x32", "train", _F32, 2, 16, 16, 32, 32, 8, 128, 1, 1, False),
        # fp32 training of a small latent model (no bf16 loss), uneven image
        _res("res-f32-24x40x128", "train", _F32, 4, 24, 40, 128, 128, 32, 512, 2, 1, False),
        # channel counts that are multiples of 32 and not of 64, odd image, small batch
        _res("res-bf16-27x45x96", "train", _BF16, 3, 27, 45, 96, 288, 32, 384, 2, 1, False),
        # the four UNet levels of an SD-like denoiser in training: the first level, one
        # microbatch of 8 latents, the overlapped decoder backward on
        _res("res-64x64x320", "train", _BF16, 8, 64, 64, 320, 320, 32, 1280, 2, 1, True),
        # the second level, whose first block widens 320 to 640 channels
        _res("res-32x32x640", "train", _BF16, 8, 32, 32, 320, 640, 32, 1280, 2, 1, True),
        # the third and fourth level: small images, weights dominate; two microbatches
        # through the schedule executor, and a small-memory microbatch of 2 latents
        _res("res-16x16x1280", "train", _BF16, 8, 16, 16, 1280, 1280, 32, 1280, 2, 2, False),
        _res("res-8x8x1280", "train", _BF16, 2, 8, 8, 1280, 1280, 32, 1280, 2, 1, False),
        # sampling with classifier-free guidance: two latents, forward only
        _res("res-sample-64x64x320", "sample", _BF16, 2, 64, 64, 320, 320, 32, 1280, 2, 1, False),
        # UViT-like training step: 256 tokens of 768 channels
        _tok("tok-256x768", "train", 16, 256, 12, 4, 2, 1, True),
        # UViT-like sampling with classifier-free guidance
        _tok("tok-sample-256x768", "sample", 2, 256, 12, 4, 2, 1, False),
        # Hunyuan-DiT-like training step: 1024 tokens of 1408 channels
        _tok("tok-1024x1408", "train", 8, 1024, 22, 4, 1, 1, True),
        # high resolution: the longest sequences the stage takes, narrow, two microbatches
        _tok("tok-4096x512", "train", 1, 4096, 8, 4, 1, 2, False),
    ]


def draw(rng):
    most = max(work(c)["flops"] for c in listed())
    while True:
        case = _draw(rng)
        w = work(case)
        if w["flops"] <= most and w["bytes"] <= 2.5e9:
            return case


def _log_int(rng, lo, hi, step=1):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def _draw(rng):
    mode = rng.choice(("train", "train", "sample"))
    micro = rng.choice((1, 1, 2)) if mode == "train" else 1
    overlap = mode == "train" and micro == 1 and rng.random() < 0.5
    if rng.random() < 0.6:
        dtype = rng.choice((_BF16, _BF16, _BF16, _F32))
        blocks = rng.choice((1, 2))
        temb = rng.choice((128, 320, 512, 1280))
        if dtype == _F32:
            c = 32 * _log_int(rng, 1, 6)
        else:
            c = 32 * _log_int(rng, 3, 40)
        cin = 32 * rng.randint(1, c // 32) if blocks == 2 and rng.random() < 0.4 else c
        groups = rng.choice((8, 16, 32))
        height = _log_int(rng, 7, 72)
        width = height if rng.random() < 0.5 else _log_int(rng, 7, 72)
        batch = _log_int(rng, 1, 16)
        return _res(None, mode, dtype, batch, height, width, cin, c, groups, temb, blocks, micro,
                    overlap)
    heads = _log_int(rng, 2, 24)
    tokens = _log_int(rng, 64, 4096, 64)
    batch = _log_int(rng, 1, 16)
    return _tok(None, mode, batch, tokens, heads, rng.choice((2, 4)), rng.choice((1, 2)), micro,
                overlap)


# ---- descriptors -------------------------------------------------------------


def _desc(case):
    if case["kind"] == "tok":
        return dict(kind="transformer", batch=case["batch"], tokens=case["tokens"],
                    width=64 * case["heads"], heads=case["heads"], eps=1e-5, mlp=case["mlp"],
                    n_enc=case["blocks"], n_dec=case["blocks"], dtype=case["dtype"],
                    max_inflight=case["micro"])
    n, c, cin = case["blocks"], case["c"], case["cin"]
    if cin == c:  # every encoder output is a skip
        enc = [dict(c_in=c, c_out=c, skip_slot_out=k) for k in range(n)]
        dec = [dict(c_up=c, c_skip=c, c_out=c, skip_slot_in=n - 1 - k) for k in range(n)]
        slot = -1
    else:  # the widening level: the last decoder block reads the stage input
        enc = [dict(c_in=cin, c_out=c, skip_slot_out=-1), dict(c_in=c, c_out=c, skip_slot_out=0)]
        dec = [dict(c_up=c, c_skip=c, c_out=c, skip_slot_in=0),
               dict(c_up=c, c_skip=cin, c_out=c, skip_slot_in=1)]
        slot = 1
    # c_up + c_skip != c_out always holds: both sources have channels
    return dict(batch=case["batch"], height=case["height"], width=case["width"],
                groups=case["groups"], eps=1e-5, temb_dim=case["temb"], dtype=case["dtype"],
                enc=enc, dec=dec, input_skip_slot=slot, max_inflight=case["micro"])


def _param_shapes(case, desc):
    return configs.tparam_names(desc) if case["kind"] == "tok" else configs.param_names(desc)


def _boundary_shapes(case):
    b = case["batch"]
    if case["kind"] == "tok":
        s = (b, case["tokens"], 64 * case["heads"])
        return dict(x=s, u=s, g_enc=s, g_dec=s)
    hw = (b, case["height"], case["width"])
    return dict(x=hw + (case["cin"],), u=hw + (case["c"],), temb=(b, case["temb"]),
                g_enc=hw + (case["c"],), g_dec=hw + (case["c"],))


def work(case):
    desc = _desc(case)
    params = sum(math.prod(s) for _, s in _param_shapes(case, desc))
    esz = 2 if case["dtype"] == _BF16 else 4
    sh = _boundary_shapes(case)
    n = {k: math.prod(s) for k, s in sh.items()}
    if case["kind"] == "tok":
        t, c, r = case["batch"] * case["tokens"], 64 * case["heads"], 64 * case["heads"] * case["mlp"]
        blk = 2.0 * t * (4 * c * c + 2 * r * c)
        att = 4.0 * t * case["tokens"] * c
        fwd = 2 * case["blocks"] * (blk + att) + case["blocks"] * 4.0 * t * c * c
    else:
        p = case["batch"] * case["height"] * case["width"]
        fwd = 0.0
        for b in desc["enc"] + desc["dec"]:
            ci = b["c_in"] if "c_in" in b else b["c_up"] + b["c_skip"]
            co = b["c_out"]
            fwd += 2.0 * p * co * 9 * (ci + co) + 2.0 * case["batch"] * co * case["temb"]
            if ci != co:
                fwd += 2.0 * p * co * ci
    if case["mode"] == "sample":
        # the weights as the stage keeps them, the inputs and both outputs
        out = n["g_enc"] + n["g_dec"]
        return dict(bytes=float(esz * (params + n["x"] + n["u"] + n.get("temb", 0) + out)),
                    flops=fwd)
    # masters read and gradients written once (fp32); per microbatch the
    # inputs and output gradients read, the outputs and input gradients written
    act = esz * (sum(n.values()) + n["g_enc"] + n["g_dec"] + n["x"] + n["u"]) + 4 * n.get("temb", 0)
    return dict(bytes=float(8 * params + case["micro"] * act), flops=3.0 * fwd * case["micro"])


def tolerance(case):
    # Against exact() over these ranges the worst output is off by 7.3e-3
    # (LayerNorm gains; 5.5e-3 for the ResBlock stage) in bf16 and 1.4e-6 in
    # fp32, its worst value by 7.5e-2 and 9.6e-6: about three to four times that.
    if case["dtype"] == _BF16:
        return {"rel": 2.5e-2, "max": 0.3}
    return {"rel": 6e-6, "max": 4e-5}


# ---- inputs --------------------------------------------------------------------


def _inputs(case, seed):
    """Parameters (name -> fp32 tensor) and per-microbatch boundary tensors,
    bf16-representable for bf16 stages."""
    dev = "cuda"
    dt = torch.bfloat16 if case["dtype"] == _BF16 else torch.float32
    gen = torch.Generator(device=dev).manual_seed(seed)

    def normal(shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=torch.float32)

    params, fan = {}, {}
    for name, shape in _param_shapes(case, _desc(case)):
        blk, leaf = name.split(".", 1)
        z = normal(shape)
        if len(shape) > 1:  # a weight: variance 1 / fan-in, its bias alike
            fan[blk] = math.prod(shape[1:])
            v = z / math.sqrt(fan[blk])
        elif leaf in ("g1", "g2", "ln1.g", "ln2.g"):
            v = 1.0 + 0.1 * z
        elif leaf in ("be1", "be2", "ln1.b", "ln2.b"):
            v = 0.1 * z
        else:
            v = z / math.sqrt(fan[blk])
        params[name] = v.to(dt).float()
    bounds = [{k: normal(s).to(dt) for k, s in _boundary_shapes(case).items()}
              for _ in range(case["micro"])]
    return params, bounds


def prepare(case, seed):
    desc = _desc(case)
    tok = case["kind"] == "tok"
    params, bounds = _inputs(case, seed)
    st = T.TStage(desc) if tok else S.Stage(desc)
    grads = {}
    for name, (off, shape) in st.layout.items():
        k = math.prod(shape)
        st.params[off:off + k].copy_(params[name].reshape(-1))
        grads[name] = st.grads[off:off + k].view(shape)
    st.sync_params()
    st.overlap_bwd(case["overlap"])
    dt = torch.bfloat16 if case["dtype"] == _BF16 else torch.float32
    io = []
    for b in bounds:
        m = dict(b)
        m["y_enc"] = torch.empty(b["g_enc"].shape, dtype=dt, device="cuda")
        m["y_dec"] = torch.empty(b["g_dec"].shape, dtype=dt, device="cuda")
        if case["mode"] == "train":
            m["dx"] = torch.empty(b["x"].shape, dtype=dt, device="cuda")
            m["du"] = torch.empty(b["u"].shape, dtype=dt, device="cuda")
            if not tok:
                m["dtemb"] = torch.zeros(b["temb"].shape, dtype=torch.float32, device="cuda")
        io.append(m)
    table = S.sched_build(1, case["micro"])[0] if case["micro"] > 1 else None
    return dict(case=case, st=st, io=io, grads=grads, table=table, tok=tok)


# ---- the pass -------------------------------------------------------------------


def _forward(st, tok, m):
    if tok:
        st.forward(T.ENC, 0, m["x"], out=m["y_enc"])
        st.forward(T.DEC, 0, m["u"], out=m["y_dec"])
    else:
        st.forward(S.ENC, 0, m["x"], m["temb"], out=m["y_enc"])
        st.forward(S.DEC, 0, m["u"], m["temb"], out=m["y_dec"])


def run(state):
    case, st, io, tok = state["case"], state["st"], state["io"], state["tok"]
    if case["mode"] == "sample":
        _forward(st, tok, io[0])
        st.release(0)
        return {"y_enc": io[0]["y_enc"], "y_dec": io[0]["y_dec"]}
    st.zero_grads()
    st.sync_params()
    for m in io:
        if not tok:
            m["dtemb"].zero_()
    if state["table"] is not None:
        step = T.tsched_run_device if tok else S.sched_run_device
        step(st, 1, 0, len(io), state["table"], io)
    else:
        m = io[0]
        _forward(st, tok, m)
        if tok:
            st.backward(T.DEC, 0, m["g_dec"], din=m["du"])
            st.backward(T.ENC, 0, m["g_enc"], din=m["dx"])
        else:
            st.backward(S.DEC, 0, m["g_dec"], din=m["du"], dtemb=m["dtemb"])
            st.backward(S.ENC, 0, m["g_enc"], din=m["dx"], dtemb=m["dtemb"])
    out = dict(state["grads"])
    for i, m in enumerate(io):
        for k in ("y_enc", "y_dec", "dx", "du", "dtemb"):
            if k in m:
                out["%s%d" % (k, i)] = m[k]
    return out


# ---- the definition in float64 ----------------------------------------------------


def _conv3(x, w):
    b, h, wd, _ = x.shape
    xp = F.pad(x, (0, 0, 1, 1, 1, 1))
    cols = torch.cat([xp[:, i:i + h, j:j + wd] for i in range(3) for j in range(3)], dim=-1)
    return (cols.reshape(b * h * wd, -1) @ w.reshape(w.shape[0], -1).t()).reshape(b, h, wd, -1)


def _gn_silu(x, g, be, groups):
    b, h, w, c = x.shape
    v = x.reshape(b, h * w, groups, c // groups)
    mean = v.mean(dim=(1, 3), keepdim=True)
    var = ((v - mean) ** 2).mean(dim=(1, 3), keepdim=True)
    z = ((v - mean) / torch.sqrt(var + 1e-5)).reshape(b, h, w, c) * g + be
    return z * torch.sigmoid(z)


def _resblock(p, k, x, temb, groups):
    e = (temb * torch.sigmoid(temb)) @ p[k + ".Wl"].t() + p[k + ".bl"] + p[k + ".b1"]
    h = _conv3(_gn_silu(x, p[k + ".g1"], p[k + ".be1"], groups), p[k + ".W1"]) + e[:, None, None]
    y = _conv3(_gn_silu(h, p[k + ".g2"], p[k + ".be2"], groups), p[k + ".W2"]) + p[k + ".b2"]
    if k + ".Ws" in p:
        return y + x @ p[k + ".Ws"].t() + p[k + ".bs"]
    return y + x


def _ln(x, g, b):
    mean = x.mean(dim=-1, keepdim=True)
    var = ((x - mean) ** 2).mean(dim=-1, keepdim=True)
    return (x - mean) / torch.sqrt(var + 1e-5) * g + b


def _tblock(p, k, x, heads):
    b, l, c = x.shape
    a = _ln(x, p[k + ".ln1.g"], p[k + ".ln1.b"])
    qkv = (a @ p[k + ".qkv.W"].t() + p[k + ".qkv.b"]).reshape(b, l, 3, heads, 64)
    q, kk, v = (qkv[:, :, i].permute(0, 2, 1, 3).contiguous() for i in range(3))
    o = torch.cat([torch.softmax(q[i] @ kk[i].transpose(1, 2).contiguous() / 8.0, dim=-1) @ v[i]
                   for i in range(b)]).reshape(b, heads, l, 64)
    h = x + o.permute(0, 2, 1, 3).reshape(b, l, c) @ p[k + ".proj.W"].t() + p[k + ".proj.b"]
    z = _ln(h, p[k + ".ln2.g"], p[k + ".ln2.b"]) @ p[k + ".fc1.W"].t() + p[k + ".fc1.b"]
    m = 0.5 * z * (1.0 + torch.erf(z / math.sqrt(2.0)))
    return h + m @ p[k + ".fc2.W"].t() + p[k + ".fc2.b"]


def _model(case, desc, p, b):
    """(y_enc, y_dec) of one microbatch in the dtype of its inputs."""
    n = case["blocks"]
    if case["kind"] == "tok":
        skips, x = [], b["x"]
        for k in range(n):
            x = _tblock(p, "enc%d" % k, x, case["heads"])
            skips.append(x)
        v = b["u"]
        for k in range(n):
            key = "dec%d" % k
            v = torch.cat([v, skips[n - 1 - k]], dim=-1) @ p[key + ".skip.W"].t() + p[key + ".skip.b"]
            v = _tblock(p, key, v, case["heads"])
        return x, v
    slots, x = {}, b["x"]
    if desc["input_skip_slot"] >= 0:
        slots[desc["input_skip_slot"]] = x
    for k, e in enumerate(desc["enc"]):
        x = _resblock(p, "enc%d" % k, x, b["temb"], case["groups"])
        if e["skip_slot_out"] >= 0:
            slots[e["skip_slot_out"]] = x
    v = b["u"]
    for k, d in enumerate(desc["dec"]):
        v = torch.cat([v, slots[d["skip_slot_in"]]], dim=-1)
        v = _resblock(p, "dec%d" % k, v, b["temb"], case["groups"])
    return x, v


def exact(case, seed):
    desc = _desc(case)
    params, bounds = _inputs(case, seed)
    train = case["mode"] == "train"
    p = {k: v.double().requires_grad_(train) for k, v in params.items()}
    out = {}
    for i, bound in enumerate(bounds):
        b = {k: v.double().requires_grad_(train and not k.startswith("g_"))
             for k, v in bound.items()}
        y_enc, y_dec = _model(case, desc, p, b)
        if not train:
            return {"y_enc": y_enc, "y_dec": y_dec}
        # one backward: the skip gradients reach the encoder through its outputs
        torch.autograd.backward([y_enc, y_dec], [b["g_enc"], b["g_dec"]])
        out["y_enc%d" % i], out["y_dec%d" % i] = y_enc.detach(), y_dec.detach()
        out["dx%d" % i], out["du%d" % i] = b["x"].grad, b["u"].grad
        if "temb" in b:
            out["dtemb%d" % i] = b["temb"].grad
    out.update({k: v.grad for k, v in p.items()})
    return out
