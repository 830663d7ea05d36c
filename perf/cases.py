"""The work a user of this library has it do, as cases to be timed: decoding shading queries
(every precision, both filters, learned frames, the albedo head), drawing samples, one training
step and the gradients behind it, the encoder's phase, and the request loop.

Every input is drawn on the device from the seed.  The sizes are those of the workloads, tests
and benchmark of this repository (a 64^2 x 8 material with 4096 queries up to a 3840 x 2160
frame; 2^20-sample training batches; the decoders 2 x 16, 2 x 32 and 3 x 64), with ragged ones
between them.
"""
import math

import numpy as np
import torch

from paper_2305_02678_amd import nam

_PRECISION = {"fp32": nam.F32, "fp16": nam.F16, "fp8": nam.FP8_E4M3}
_contexts = {}


def _context(deterministic=False):
    """One context per process, as a user's program has (another one for the reproducible mode)."""
    if deterministic not in _contexts:
        _contexts[deterministic] = nam.Context(0)
        _contexts[deterministic].set_deterministic(deterministic)
    return _contexts[deterministic]


def _case(name, kind, n, tex=2048, channels=16, hidden=64, layers=3, frames=0, albedo=False, precision="fp32",
          stochastic=False, clamp=False, deterministic=False):
    c = dict(kind=kind, n=n, tex=tex, channels=channels, hidden=hidden, layers=layers, frames=frames, albedo=albedo,
             precision=precision, stochastic=stochastic, clamp=clamp, deterministic=deterministic)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest request a renderer or the request loop sends: launch latency
        _case("decode_tile_fp16", "decode", 4096, precision="fp16"),
        # one 1080p frame, the benchmark's workload, in the precision that is deployed
        _case("decode_frame_fp16", "decode", 1920 * 1080, precision="fp16"),
        # the same frame in full precision: previews of a material in training, references
        _case("decode_frame_fp32", "decode", 1920 * 1080),
        # lowest precision with the albedo head, clamped atlas texture, a ragged laptop screen
        _case("decode_albedo_fp8", "decode", 1366 * 768 - 11, tex=1024, albedo=True, precision="fp8", clamp=True),
        # the paper's setting at 4k: learned frames and the stochastic level choice
        _case("decode_framed_4k_fp16", "decode", 3840 * 2160, frames=2, precision="fp16", stochastic=True),
        # an odd wavefront of a path tracer in full precision, the paper's middle decoder (2 x 32)
        _case("decode_framed_odd_fp32", "decode", 500009, tex=1024, channels=8, hidden=32, layers=2, frames=2,
              stochastic=True),
        # importance sampling: one direction and its density per pixel
        _case("sample_frame_fp16", "sample", 1920 * 1080, precision="fp16"),
        # one step of training texels and decoder (loss, gradients, Adam) on a 2^20 batch
        _case("train_step", "train", 1 << 20, tex=1024),
        # gradients for a user's own optimiser with two learned frames, a ragged batch
        _case("gradients_framed", "loss", 250007, tex=1024, frames=2),
        # a small batch through torch.autograd with the paper's smallest decoder (2 x 16)
        _case("autograd_small", "autograd", 16384, tex=256, channels=8, hidden=16, layers=2, clamp=True),
        # one step of the encoder's phase: codes, loss on them, both gradients
        _case("encoder_step", "encoder", 1 << 20, tex=1024),
        # the request loop: requests of mixed sizes over several resident materials
        _case("serve_mixed_fp16", "serve", 2400000, tex=1024, precision="fp16"),
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    hidden, layers = rng.choice([(16, 2), (32, 2), (32, 3), (64, 2), (64, 3), (64, 3)])
    shape = dict(tex=rng.choice([256, 512, 1024, 2048]), channels=rng.choice([8, 16]), hidden=hidden, layers=layers,
                 clamp=rng.random() < 0.25)
    kind = rng.choice(["decode"] * 4 + ["sample", "pdf", "train", "loss", "autograd", "encoder", "serve"])
    if kind == "decode":
        precision = rng.choice(["fp32", "fp16", "fp16", "fp8"])
        n = _log_int(rng, 4096, 1920 * 1080 if precision == "fp32" else 3840 * 2160)
        return _case(None, kind, n, frames=rng.choice([0, 0, 1, 2]), albedo=rng.random() < 0.25, precision=precision,
                     stochastic=rng.random() < 0.4, **shape)
    if kind in ("sample", "pdf"):
        return _case(None, kind, _log_int(rng, 4096, 1920 * 1080), precision=rng.choice(["fp32", "fp16", "fp16"]),
                     **shape)
    if kind == "serve":
        return _case(None, kind, _log_int(rng, 200000, 4000000), precision=rng.choice(["fp32", "fp16", "fp8"]), **shape)
    shape["tex"] = min(shape["tex"], 1024)
    if kind == "encoder":
        return _case(None, kind, _log_int(rng, 8192, 1 << 20), **shape)
    # training: 2 x 16 and framed decoders are cheap to hold and are met in smaller batches
    frames = rng.choice([0, 0, 2]) if hidden > 16 else 0
    n = _log_int(rng, 8192, 250007 if frames or hidden == 16 else 1 << 20)
    return _case(None, kind, n, frames=frames, albedo=not frames and rng.random() < 0.25,
                 deterministic=kind == "loss" and rng.random() < 0.3, **shape)


# ---- inputs


def _dims(c):
    return [c["channels"] + 6 * max(1, c["frames"])] + [c["hidden"]] * c["layers"] + [6 if c["albedo"] else 3]


def _levels(tex):
    return int(math.log2(tex)) + 1


def _texels(tex):
    return sum(max(1, tex >> l) ** 2 for l in range(_levels(tex)))


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


class _Draw:
    """Seeded draws on the device."""

    def __init__(self, case, seed):
        self.g = torch.Generator(device=_device())
        self.g.manual_seed(1000003 * seed + case["n"])

    def rand(self, *shape):
        return torch.rand(shape, generator=self.g, device=self.g.device)

    def randn(self, *shape):
        return torch.randn(shape, generator=self.g, device=self.g.device)

    def mlp(self, dims):
        """Xavier weights with small biases, packed W_1, b_1, W_2, ..."""
        out = []
        for fi, fo in zip(dims, dims[1:]):
            out.append((2 * self.rand(fo * fi) - 1) * math.sqrt(6.0 / (fi + fo)))
            out.append(0.1 * self.randn(fo))
        return torch.cat(out)

    def frame_layer(self, frames, channels):
        """Normals about +z and tangents about +x, steered by the latent code."""
        w = 0.25 * (2 * self.rand(6 * frames * channels) - 1) * math.sqrt(6.0 / (channels + 6 * frames))
        b = torch.tensor([0.0, 0.0, 1.0, 1.0, 0.0, 0.0] * frames, device=w.device)
        return torch.cat([w, b])

    def pyramid(self, level0):
        out = [level0]
        while out[-1].shape[0] > 1:
            p = out[-1]
            p = 0.5 * (p[0::2] + p[1::2])
            out.append((0.5 * (p[:, 0::2] + p[:, 1::2])).contiguous())
        return out

    def directions(self, n):
        """Cosine-distributed on the upper hemisphere."""
        a, b = self.rand(n), self.rand(n)
        r, phi = a.sqrt(), 2 * math.pi * b
        return torch.stack([r * phi.cos(), r * phi.sin(), (1 - a).sqrt()], 1).contiguous()

    def screen(self, n, tex):
        """n pixels of a 16:9 frame in 16 x 16 screen tiles, a smooth affine map with a warp onto
        the texture and the level of the pixel's footprint."""
        k = self.rand(12).double().cpu().numpy()
        w = int(math.ceil(math.sqrt(n * 16.0 / 9.0)))
        h = int(math.ceil(n / w))
        dev = self.g.device
        y, x = torch.meshgrid(torch.arange(h, device=dev), torch.arange(w, device=dev), indexing="ij")
        key = ((y // 16) * ((w + 15) // 16) + x // 16) * 256 + (y % 16) * 16 + x % 16
        order = key.reshape(-1).argsort()[:n]
        x, y = (t.reshape(-1)[order].double() + 0.5 for t in (x, y))
        th, sh = 2 * math.pi * k[0], 0.4 * k[1] - 0.2
        kx, ky = (0.7 * (12 / 0.7) ** v / tex for v in k[2:4])
        A = np.array([[math.cos(th), -math.sin(th)], [math.sin(th), math.cos(th)]]) @ np.diag([kx, ky]) @ np.array(
            [[1.0, sh], [0.0, 1.0]])
        au, av = 2 * math.pi * int(1 + 3 * k[4]) / w, 2 * math.pi * int(1 + 3 * k[5]) / h
        pu, pv = 2 * math.pi * k[6], 2 * math.pi * k[7]
        u = A[0, 0] * x + A[0, 1] * y + k[8] + 0.02 * torch.sin(au * x + pu)
        v = A[1, 0] * x + A[1, 1] * y + k[9] + 0.02 * torch.sin(av * y + pv)
        det = (A[0, 0] + 0.02 * au * torch.cos(au * x + pu)) * (A[1, 1] + 0.02 * av * torch.cos(av * y + pv)) - (
            A[0, 1] * A[1, 0])
        lod = 0.5 * torch.log2((det.abs() * tex * tex).clamp_min(1e-30))
        return torch.stack([u, v], 1).float().contiguous(), lod.float().contiguous()

    def batch(self, n, tex):
        """Training samples: uv uniform, level Exp(1) truncated to the pyramid."""
        hi = _levels(tex) - 1
        return self.rand(n, 2), -torch.log1p(-self.rand(n) * (1.0 - math.exp(-hi)))

    def targets(self, uv, wi, wo, outputs):
        """A spatially varying diffuse and GGX reflectance (then an albedo estimate)."""
        k = torch.arange(1, 5, device=uv.device)
        t = 2 * math.pi * (uv[:, :1] * k + uv[:, 1:] * k.flip(0))
        rho = 0.05 + 0.9 * torch.sigmoid(2 * torch.sin(t[:, :3]))
        a2 = (0.3 + 0.6 * torch.sigmoid(torch.sin(t[:, 3]))) ** 4
        h = torch.nn.functional.normalize(wi + wo, dim=1)
        d = a2 / (math.pi * (h[:, 2] ** 2 * (a2 - 1) + 1) ** 2)
        g = 1.0
        for c in (wi[:, 2], wo[:, 2]):
            g = g / (c + torch.sqrt(a2 + (1 - a2) * c * c))
        f = 0.04 + 0.96 * (1 - (wi * h).sum(1)).clamp(0, 1) ** 5
        brdf = rho / math.pi + (f * d * g)[:, None]
        return (torch.cat([brdf, rho + 0.1 * self.rand(len(uv), 3)], 1) if outputs == 6 else brdf).contiguous()


def _serve_shapes(case):
    """Four resident materials and the sizes of sixteen requests that add up to about n queries."""
    mats = [(case["tex"], case["channels"]), (512, 8), (case["tex"], 24 - case["channels"]), (256, 16)]
    share = [2.0 ** (i % 8) for i in range(16)]
    return mats, [max(4096, int(case["n"] * s / sum(share)) + 37 * i) for i, s in enumerate(share)]


def _inputs(case, seed):
    """Everything a case reads, as device tensors."""
    d, n, tex, C = _Draw(case, seed), case["n"], case["tex"], case["channels"]
    i = {}
    if case["kind"] == "serve":
        mats, sizes = _serve_shapes(case)
        i["materials"] = []
        for side, ch in mats:
            dims = [ch + 6] + _dims(case)[1:]
            i["materials"].append((d.pyramid(d.randn(side, side, ch)), dims, d.mlp(dims)))
        i["requests"] = []
        for k, m in enumerate(sizes):
            uv, lod = d.screen(m, mats[k % 4][0])
            i["requests"].append((k % 4, (uv, lod, d.directions(m), d.directions(m))))
        return i
    i["dims"] = _dims(case)
    if case["kind"] == "encoder":
        x = (torch.arange(tex, device=d.g.device) + 0.5) / tex
        f = 2 * math.pi * (d.rand(4, 2) * 4 + 1).floor()
        p = 2 * math.pi * d.rand(4)
        s = torch.sin(f[:, 0] * x[:, None, None] + f[:, 1] * x[None, :, None] + p)
        i["attrs"] = torch.cat([l.reshape(-1, 4) for l in d.pyramid(0.05 + 0.9 * torch.sigmoid(s))]).contiguous()
        i["edims"] = [4, 32, 32, C]
        i["eparams"] = d.mlp(i["edims"])
    else:
        i["levels"] = d.pyramid(d.randn(tex, tex, C))
    i["params"] = d.mlp(i["dims"])
    i["frames"] = d.frame_layer(case["frames"], C) if case["frames"] else None
    if case["kind"] in ("decode", "sample", "pdf"):
        i["uv"], i["lod"] = d.screen(n, tex)
    else:
        i["uv"], i["lod"] = d.batch(n, tex)
    i["wi"], i["wo"] = d.directions(n), d.directions(n)
    if case["kind"] in ("sample", "pdf"):
        i["sdims"] = [C + 3, 32, 32, 32, 9]
        i["sparams"] = d.mlp(i["sdims"])
        i["u"] = d.rand(n, 3)
    elif case["kind"] == "decode":
        i["xi"] = d.rand(n) if case["stochastic"] else None
    elif case["kind"] == "autograd":
        i["d_rgb"] = d.randn(n, i["dims"][-1]) / n
    else:
        i["target"] = d.targets(i["uv"], i["wi"], i["wo"], i["dims"][-1])
    return i


def _material(ctx, case, levels, dims, params, frames, calibration):
    m = nam.Material(ctx, [l.cpu().numpy() for l in levels], dims, params.cpu().numpy(),
                     nam.CLAMP if case["clamp"] else nam.WRAP, case["frames"] if frames is not None else 0,
                     None if frames is None else frames.cpu().numpy())
    if case["precision"] != "fp32":
        am = m.calibrate(*calibration) if case["precision"] == "fp8" else None
        m.set_precision(_PRECISION[case["precision"]], nam.F16, am)
    return m


def prepare(case, seed):
    ctx = _context(case["deterministic"])
    i = _inputs(case, seed)
    s = {"case": case, "ctx": ctx, "in": i}
    address = nam.CLAMP if case["clamp"] else nam.WRAP
    if case["kind"] == "serve":
        s["server"] = nam.Server(ctx)
        s["materials"] = []
        for k, (levels, dims, params) in enumerate(i["materials"]):
            m = _material(ctx, case, levels, dims, params, None, i["requests"][k][1])
            s["materials"].append((m, s["server"].add_material(m)))
        s["rgb"] = [torch.zeros(len(q[1]), _dims(case)[-1], device=q[1].device) for _, q in i["requests"]]
        i.pop("materials")
        return s
    if case["kind"] in ("decode", "sample", "pdf"):
        s["material"] = _material(ctx, case, i.pop("levels"), i["dims"], i["params"], i["frames"],
                                  (i["uv"], i["lod"], i["wi"], i["wo"]))
        if "sparams" in i:
            s["material"].set_sampler(i["sdims"], i["sparams"].cpu().numpy())
        return s
    s["model"] = nam.Model(ctx, case["tex"], case["tex"], case["channels"], _levels(case["tex"]), i["dims"], address,
                           case["frames"])
    s["params"] = i["params"] if i["frames"] is None else torch.cat([i["frames"], i["params"]])
    if case["kind"] == "encoder":
        s["encoder"] = nam.Encoder(ctx, i["edims"], case["tex"], case["tex"], _levels(case["tex"]), address)
        return s
    s["texels"] = torch.cat([l.reshape(-1, case["channels"]) for l in i.pop("levels")]).contiguous()
    if case["kind"] == "train":
        s["trainer"] = nam.Trainer(s["model"], s["texels"], s["params"])
    elif case["kind"] == "autograd":
        s["texels"].requires_grad_()
        s["params"].requires_grad_()
    return s


def run(state):
    case, i = state["case"], state["in"]
    kind = case["kind"]
    if kind == "serve":
        server = state["server"]
        for (m, q), rgb in zip(i["requests"], state["rgb"]):
            server.submit(state["materials"][m][1], *q, rgb)
        server.wait_all()
        return state["rgb"]
    q = (i["uv"], i["lod"], i["wi"], i["wo"])
    if kind == "decode":
        return nam.decode(state["material"], *q, xi=i["xi"])
    if kind == "sample":
        return nam.sampler_sample(state["material"], i["uv"], i["lod"], i["wi"], i["u"])
    if kind == "pdf":
        return nam.sampler_pdf(state["material"], *q)
    if kind == "train":
        t = state["trainer"]
        loss = t.step(*q, i["target"])
        return loss, t.texels, t.params, t.m_tex, t.m_par
    if kind == "loss":
        return state["model"].loss_backward(state["texels"], state["params"], *q, i["target"])
    if kind == "autograd":
        rgb = nam.neural_material(state["texels"], state["params"], *q, state["model"])
        grads = torch.autograd.grad(rgb, (state["texels"], state["params"]), i["d_rgb"])
        return rgb, *grads
    z = state["encoder"].encode_queries(i["eparams"], i["attrs"], i["uv"], i["lod"])
    loss, dz, d_params = state["model"].loss_backward_codes(state["params"], z, i["wi"], i["wo"], i["target"])
    return z, loss, dz, d_params, state["encoder"].backward(i["eparams"], i["attrs"], i["uv"], i["lod"], dz)


# ---- the least a pass has to move and compute


def _mlp_work(dims):
    return 2.0 * sum(a * b for a, b in zip(dims, dims[1:]))


def work(case):
    n, C, tex, dims = case["n"], case["channels"], case["tex"], _dims(case)
    size = 4 if case["precision"] == "fp32" else 2
    if case["kind"] == "serve":
        mats, sizes = _serve_shapes(case)
        read = sum(min(_texels(s), 1.25 * sum(sizes[k::4])) * c * size for k, (s, c) in enumerate(mats))
        flops = sum(m * _mlp_work([mats[k % 4][1] + 6] + dims[1:]) for k, m in enumerate(sizes))
        return {"bytes": read + sum(sizes) * (36 + 4 * dims[-1]), "flops": flops}
    if case["kind"] in ("decode", "sample", "pdf"):
        # about one texel of the finer level and a quarter of the coarser one per pixel
        read = min(_texels(tex), 1.25 * n) * C * size
        if case["kind"] == "decode":
            io = 36 + 4 * dims[-1] + (4 if case["stochastic"] else 0)
            extra = 2.0 * 6 * case["frames"] * C + 36 * case["frames"]
            return {"bytes": read + n * io, "flops": n * (_mlp_work(dims) + extra)}
        io = 52 if case["kind"] == "sample" else 40
        return {"bytes": read + n * io, "flops": n * _mlp_work([C + 3, 32, 32, 32, 9])}
    io = 36 + 4 * dims[-1]
    if case["kind"] == "encoder":
        e = _mlp_work([4, 32, 32, C])
        return {"bytes": min(_texels(tex), 8.0 * n) * 16 + n * (2 * 4 * C + io), "flops": n * (4 * e + 3 * _mlp_work(dims))}
    touched = min(_texels(tex), 8.0 * n) * C * 4
    dense = _texels(tex) * C * 4.0
    # gradients are written once; a step also reads and writes the texels and both moments
    moved = touched + (6 * dense if case["kind"] == "train" else dense)
    return {"bytes": moved + n * (io + (4 * dims[-1] if case["kind"] == "autograd" else 0)),
            "flops": 3 * n * _mlp_work(dims)}


# ---- the same results in 64 bits, in plain torch


def _taps(case, tex, uv, lod, xi=None):
    """Texel indices and weights of every query (8 taps, or the 4 of the level drawn)."""
    M = _levels(tex)
    first = torch.tensor(np.cumsum([0] + [max(1, tex >> l) ** 2 for l in range(M)])[:-1].copy(), device=uv.device)
    lam = lod.double().clamp(0, M - 1)
    l0 = lam.floor().long()
    t = lam - l0
    l1 = (l0 + 1).clamp_max(M - 1)
    which = [(l0, 1 - t), (l1, t)] if xi is None else [(torch.where(xi.double() < t, l1, l0), torch.ones_like(t))]
    idx, w = [], []
    for l, share in which:
        side = (tex >> l).clamp_min(1)
        p = uv.double() * side[:, None] - 0.5
        i = p.floor()
        a = p - i
        i = i.long()
        for dy in (0, 1):
            for dx in (0, 1):
                x, y = i[:, 0] + dx, i[:, 1] + dy
                if case["clamp"]:
                    x, y = torch.minimum(x.clamp_min(0), side - 1), torch.minimum(y.clamp_min(0), side - 1)
                else:
                    x, y = x % side, y % side
                idx.append(first[l] + y * side + x)
                w.append(share * (a[:, 0] if dx else 1 - a[:, 0]) * (a[:, 1] if dy else 1 - a[:, 1]))
    return idx, w


def _filter(texels, taps):
    return sum(w[:, None] * texels.index_select(0, i).double() for i, w in zip(*taps))


def _mlp(dims, params, x):
    o = 0
    for k, (fi, fo) in enumerate(zip(dims, dims[1:])):
        W, b = params[o:o + fi * fo].reshape(fo, fi), params[o + fi * fo:o + fi * fo + fo]
        o += fi * fo + fo
        x = x @ W.T + b
        x = x.relu() if k < len(dims) - 2 else x
    return x


def _softplus(x):
    return x.clamp_min(0) + torch.log1p(torch.exp(-x.abs()))


def _decoder_input(case, z, wi, wo, frames):
    """[z, T wi, T wo]; the frame layer gives a normal and a tangent per frame, each normalised."""
    wi, wo = wi.double(), wo.double()
    if frames is None:
        return torch.cat([z, wi, wo], 1)
    nf, C = case["frames"], case["channels"]
    v = z @ frames[:6 * nf * C].reshape(6 * nf, C).T + frames[6 * nf * C:]

    def unit(a):
        return a * (a * a).sum(1, keepdim=True).clamp_min(1e-12).rsqrt()

    rows = []
    for f in range(nf):
        nrm, tan = unit(v[:, 6 * f:6 * f + 3]), unit(v[:, 6 * f + 3:6 * f + 6])
        rows += [tan, unit(torch.linalg.cross(nrm, tan)), nrm]
    return torch.cat([z] + [torch.stack([(r * d).sum(1) for r in rows], 1) for d in (wi, wo)], 1)


def _decode64(case, tex, texels, dims, params, frames, q, xi=None):
    out = []
    for a in range(0, len(q[1]), 1 << 19):
        uv, lod, wi, wo = (t[a:a + (1 << 19)] for t in q)
        z = _filter(texels, _taps(case, tex, uv, lod, None if xi is None else xi[a:a + (1 << 19)]))
        out.append(_softplus(_mlp(dims, params, _decoder_input(case, z, wi, wo, frames))))
    return torch.cat(out)


def _proxy(o):
    """The sampling proxy's parameters from the network's nine outputs."""
    def qtanh(x):
        return torch.where(x.abs() < 2, x * (1 - x.abs() / 4), x.sign())

    def qsinh(x):
        return x * (1 + x.abs() / 2)

    w = torch.softmax(o[:, [0, 3]], 1)
    alpha = 1e-3 + (1 - 1e-3) * (1 + qtanh(o[:, 4:6])) / 2
    return w[:, 0], w[:, 1], qsinh(o[:, 1:3]), alpha, 0.999 * qtanh(o[:, 6]), qsinh(o[:, 7:9])


def _pdf64(p, wi, wo):
    wd, ws, mu_d, al, rho, mu_s = p
    nd = torch.nn.functional.normalize(torch.cat([-mu_d, torch.ones_like(mu_d[:, :1])], 1), dim=1)
    h = torch.nn.functional.normalize(wi + wo, dim=1)
    h = torch.where(h[:, 2:] < 0, -h, h)
    sq = torch.sqrt(1 - rho * rho)
    x = (h[:, 0] + mu_s[:, 0] * h[:, 2]) / al[:, 0]
    y = ((h[:, 1] + mu_s[:, 1] * h[:, 2]) / al[:, 1] - rho * x) / sq
    m2 = x * x + y * y + h[:, 2] ** 2
    spec = h[:, 2].clamp_min(0) / (math.pi * m2 * m2) / (al[:, 0] * al[:, 1] * sq) / (4 * (wo * h).sum(1).abs())
    return wd * (wo * nd).sum(1).clamp_min(0) / math.pi + ws * spec


def exact(case, seed):
    i, tex, kind = _inputs(case, seed), case["tex"], case["kind"]
    if kind == "serve":
        out = []
        for m, q in i["requests"]:
            levels, dims, params = i["materials"][m]
            texels = torch.cat([l.reshape(-1, l.shape[-1]) for l in levels])
            out.append(_decode64(case, levels[0].shape[0], texels, dims, params.double(), None, q))
        return out
    params = i["params"].double()
    frames = None if i["frames"] is None else i["frames"].double()
    q = (i["uv"], i["lod"], i["wi"], i["wo"])
    texels = torch.cat([l.reshape(-1, l.shape[-1]) for l in i["levels"]]) if "levels" in i else None
    if kind == "decode":
        return _decode64(case, tex, texels, i["dims"], params, frames, q, i["xi"])
    if kind in ("sample", "pdf"):
        z = _filter(texels, _taps(case, tex, i["uv"], i["lod"]))
        p = _proxy(_mlp(i["sdims"], i["sparams"].double(), torch.cat([z, i["wi"].double()], 1)))
        if kind == "pdf":
            # a half-precision sampler's density at a narrow lobe is not the exact one's
            return _pdf64(p, i["wi"].double(), i["wo"].double()) if case["precision"] == "fp32" else None
        return None  # which lobe a draw takes is decided by the last bits of its weight
    if kind == "encoder":
        attrs, eparams = i["attrs"].double(), i["eparams"].double().requires_grad_()
        params.requires_grad_()
        z = _mlp(i["edims"], eparams, _filter(attrs, _taps(case, tex, i["uv"], i["lod"])))
        # the same rounding of the codes as between the calls
        zr = z.detach().float().double().requires_grad_()
        rgb = _softplus(_mlp(i["dims"], params, _decoder_input(case, zr, i["wi"], i["wo"], None)))
        loss = ((rgb - i["target"].double()) ** 2).sum() / (3 * case["n"])
        dz, d_params = torch.autograd.grad(loss, (zr, params))
        d_eparams, = torch.autograd.grad(z, eparams, dz)
        return z.detach(), loss.detach().reshape(1), dz, d_params, d_eparams
    texels = texels.double().requires_grad_()
    p = (params if frames is None else torch.cat([frames, params])).requires_grad_()
    nf = 0 if frames is None else frames.numel()
    z = _filter(texels, _taps(case, tex, i["uv"], i["lod"]))
    rgb = _softplus(_mlp(i["dims"], p[nf:], _decoder_input(case, z, i["wi"], i["wo"], p[:nf] if nf else None)))
    if kind == "autograd":
        return rgb.detach(), *torch.autograd.grad(rgb, (texels, p), i["d_rgb"].double())
    loss = ((rgb - i["target"].double()) ** 2).sum() / (3 * case["n"])
    g = torch.autograd.grad(loss, (texels, p))
    loss = loss.detach().reshape(1)
    if kind == "loss":
        return loss, *g
    # the first Adam step from zero moments
    new = [(x.detach() - 1e-3 * gx / (gx.abs() + 1e-8)) for x, gx in zip((texels, p), g)]
    return loss, new[0], new[1], 0.1 * g[0], 0.1 * g[1]
