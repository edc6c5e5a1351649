"""Timing cases of the reconstruction library: what a user's program has it do.

Each case is one call pattern through the public Python entry points
(AltGDmin, WsInit) at one problem shape.  The kinds (`op`):

  recon   a whole reconstruction: bind the data, spectral initialisation,
          `iters` iterations, the images of the last iterate
  steps   a few iterations from a given basis on a bound problem: a
          mini-batch of the subspace tracker, a continued run
  init    the spectral initialisation and the first LS step, and the images
          they give (the first reconstruction a user sees)
  online  one new frame of the online tracker with the mean image and the
          basis fixed: residual, LS step, residual, per-frame CGLS, output
  mean    the mean image by conjugate gradients
  mec1    the modelling error by three CGLS iterations per frame
  mec2    the modelling error by ISTA on the temporal DFT
  ops     the measurement operator and its adjoint
  cnn     one training step's gradients of the warm-start network

Masks: "lines" (variable-density phase-encode lines, eight centre lines in
every frame, `lines` of them per frame; `ragged` frames hold between three
quarters of them and all) and "radial" (`spokes` golden-angle spokes per
frame rounded onto the grid).  Sequences are a body with static organs, a
moving, changing heart and a few regions with uptake curves, under a smooth
phase, with 1 % of the pixels off by a little and noise at 30 dB.
"""
import math

import numpy as np
import torch

import paper_2212_09664_amd as ag

DEV = "cuda:0"
GOLDEN = math.pi * (math.sqrt(5.0) - 1.0) / 2.0  # the golden angle, in radians


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _case(op, nx, ny, nc, q, r, mask="lines", lines=0, spokes=0, ragged=False, mixed=False, iters=0, batch=0,
          name=None):
    c = dict(op=op, nx=nx, ny=ny, nc=nc, q=q, r=r, mask=mask, lines=lines, spokes=spokes, ragged=ragged,
             mixed=mixed, iters=iters, batch=batch)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one frame of an online scan: the smallest call, bound by launches and latency
        _case("online", 128, 128, 8, 1, 6, lines=16, name="online_frame_128"),
        # a small whole reconstruction (a preview, a simulation study)
        _case("recon", 64, 64, 4, 16, 4, lines=16, iters=20, name="recon_64"),
        # the cardiac cine sequence reconstructed from start to end
        _case("recon", 256, 256, 12, 40, 8, lines=32, iters=70, name="recon_cine_256"),
        # a mini-batch of a radial perfusion scan, rank 10, general mask
        _case("steps", 128, 128, 8, 100, 10, mask="radial", spokes=16, iters=5, name="steps_radial_128"),
        # the high-rank cine sequence: rank 16, 16 coils, 64 frames
        _case("steps", 256, 256, 16, 64, 16, lines=21, iters=5, name="steps_cine_256_r16"),
        # the mixed-precision form, odd sizes and frames of unequal length
        _case("steps", 256, 256, 11, 37, 7, lines=32, ragged=True, mixed=True, iters=5, name="steps_mixed_256"),
        # the start of a long radial scan: 100 frames in the eigenproblem
        _case("init", 128, 128, 8, 100, 10, mask="radial", spokes=16, name="init_radial_128"),
        # the mean image of the cine sequence
        _case("mean", 256, 256, 12, 40, 8, lines=32, name="mean_cine_256"),
        # modelling-error correction, both models, on either kind of mask
        _case("mec1", 128, 128, 8, 64, 8, mask="radial", spokes=16, name="mec1_radial_128"),
        _case("mec2", 128, 128, 8, 48, 6, lines=16, name="mec2_cine_128"),
        # the operators alone at the largest grid (a user's own iterative method)
        _case("ops", 512, 512, 16, 24, 4, lines=64, name="ops_512"),
        # training the warm start: 16 sequences of the 128 x 128 shape
        _case("cnn", 128, 128, 0, 48, 6, batch=16, name="cnn_grad_128"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["online", "recon", "steps", "steps", "init", "mean", "mec1", "mec2", "ops", "cnn"])
    if op == "cnn":
        nx, ny = rng.choice([32, 64, 72, 96, 128]), rng.choice([32, 64, 88, 104, 128])
        return _case("cnn", nx, ny, 0, rng.randint(9, 48), rng.randint(2, 8), batch=rng.randint(1, 16))
    mask = "radial" if rng.random() < 0.35 else "lines"
    sizes = [64, 128, 256] if op != "ops" else [64, 128, 256, 512]
    while True:
        nx, ny = rng.choice(sizes), rng.choice(sizes)
        nc, q, r = rng.randint(3, 16), _log_int(rng, 12, 100), rng.randint(3, 16)
        if op == "online":
            q = 1
        # the work of the largest listed case, and a rank the frames can carry
        if nx * ny * nc * q <= (1 << 26 if op in ("ops", "steps") else 1 << 25) and (q == 1 or r <= q // 3):
            break
    accel = rng.choice([5, 6, 7, 8, 10, 12])
    lines = max(12, round(ny / accel))
    spokes = rng.randint(12, 24)
    iters = {"recon": rng.randint(10, 40), "steps": rng.randint(3, 10)}.get(op, 0)
    mixed = op in ("recon", "steps") and rng.random() < 0.25
    ragged = mask == "lines" and op != "online" and rng.random() < 0.5
    if mask == "radial":
        lines = 0
    else:
        spokes = 0
    return _case(op, nx, ny, nc, q, r, mask, lines, spokes, ragged, mixed, iters)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _grid(nx, ny):
    xs = -1.0 + 2.0 * torch.arange(nx, device=DEV, dtype=torch.float64) / nx
    ys = -1.0 + 2.0 * torch.arange(ny, device=DEV, dtype=torch.float64) / ny
    return xs[None, :], ys[:, None]


def _ellipse(X, Y, cx, cy, ax, ay):
    rho = torch.sqrt(((X - cx) / ax) ** 2 + ((Y - cy) / ay) ** 2)
    return 1.0 / (1.0 + torch.exp(torch.clamp((rho - 1.0) / 0.02, -60.0, 60.0)))


def _coil_maps(nx, ny, nc):
    """Gaussian bumps on a ring, each with its own phase, sum |s|^2 = 1."""
    X, Y = _grid(nx, ny)
    maps = []
    for c in range(nc):
        a = 2.0 * math.pi * c / nc
        mag = torch.exp(-((X - 1.2 * math.cos(a)) ** 2 + (Y - 1.2 * math.sin(a)) ** 2) / (2.0 * 0.8 ** 2))
        maps.append(mag * complex(math.cos(a), math.sin(a)))
    m = torch.stack(maps)
    return (m / torch.sqrt((m.abs() ** 2).sum(0, keepdim=True))).reshape(nc, nx * ny).to(torch.complex64)


def _sequence(nx, ny, q, rng, gen):
    """q frames (q, n) complex128."""
    X, Y = _grid(nx, ny)
    u = lambda a, b: float(rng.uniform(a, b))  # noqa: E731
    body = 0.6 * _ellipse(X, Y, u(-.05, .05), u(-.05, .05), u(.7, .8), u(.55, .65))
    static = body + 0.8 * _ellipse(X, Y, -0.35, 0.2, u(.12, .18), u(.2, .3))
    static = static + 0.4 * _ellipse(X, Y, 0.35, -0.25, u(.17, .23), u(.1, .14))
    regions = []
    for _ in range(12):
        shape = _ellipse(X, Y, u(-.5, .5), u(-.45, .45), u(.06, .2), u(.06, .2))
        f, ph = u(0.2, 1.0) * max(q, 8) / 20.0, u(0, 2 * math.pi)
        regions.append((shape, [u(.8, 1.2) * math.cos(2 * math.pi * f * k / max(q, 8) + ph) for k in range(q)], u(.2, .5)))
    ph0, cx, cy = u(0, 2 * math.pi), u(0, .2), u(-.05, .15)
    phase = torch.exp(1j * math.pi * 0.25 * (X + Y))
    n = nx * ny
    Z = torch.empty(q, n, dtype=torch.complex128, device=DEV)
    for k in range(q):
        t = 2.0 * math.pi * k / 20.0 + ph0
        s = 1.0 + 0.2 * math.sin(t)
        img = static + (1.0 + 0.15 * math.cos(t)) * _ellipse(X, Y, cx, cy, 0.22 * s, 0.18 * s)
        for shape, curve, amp in regions:
            img = img + amp * curve[k] * shape
        Z[k] = (img * phase).reshape(-1)
    off = torch.rand(q, n, device=DEV, generator=gen) < 0.01
    ang = 2.0 * math.pi * torch.rand(q, n, device=DEV, generator=gen, dtype=torch.float64)
    Z += 0.05 * off * torch.polar(torch.ones_like(ang), ang)
    return Z


def _masks(case, rng):
    """Per frame: the sampled lines ky, or the sampled flat k-space indices."""
    nx, ny, q = case["nx"], case["ny"], case["q"]
    out = []
    if case["mask"] == "lines":
        f = np.arange(-ny // 2, ny // 2)
        centre = f[(f >= -4) & (f < 4)]
        others = np.setdiff1d(f, centre)
        w = (1.0 - 2.0 * np.abs(others) / ny) ** 3 + 0.05
        full = case["lines"]
        for k in range(q):
            lo = (3 * full + 3) // 4
            nl = full if not case["ragged"] or k == 0 else int(rng.integers(lo, full + 1))
            pick = rng.choice(others, size=nl - len(centre), replace=False, p=w / w.sum())
            out.append(np.sort(np.mod(np.concatenate([centre, pick]), ny)).astype(np.int32))
        return out
    t = np.arange(-max(nx, ny) // 2, max(nx, ny) // 2, dtype=np.float64)
    first = 17 * q  # the scan was running before these frames (every seed sees the same trajectory)
    for k in range(q):
        th = (first + k * case["spokes"] + np.arange(case["spokes"])) * GOLDEN
        kx = np.floor(np.outer(np.cos(th), t) * (nx / max(nx, ny)) + 0.5).astype(np.int64) % nx
        ky = np.floor(np.outer(np.sin(th), t) * (ny / max(nx, ny)) + 0.5).astype(np.int64) % ny
        out.append(np.unique(ky * nx + kx).astype(np.int32))
    return out


def _flat(case, masks):
    """Per frame: the flat k-space indices in the measurement layout's order."""
    if case["mask"] == "lines":
        return [torch.from_numpy((l[:, None].astype(np.int64) * case["nx"] + np.arange(case["nx"])).reshape(-1)).to(DEV)
                for l in masks]
    return [torch.from_numpy(m.astype(np.int64)).to(DEV) for m in masks]


def _forward(case, coils, idx, Z, m_max):
    """y[k, c, i] = F(s_c z_k) at the frame's samples, in 64 bits."""
    nc, ny, nx = case["nc"], case["ny"], case["nx"]
    y = torch.zeros(case["q"], nc, m_max, dtype=torch.complex128, device=DEV)
    for k in range(case["q"]):
        img = (coils * Z[k][None, :]).reshape(nc, ny, nx)
        y[k, :, :idx[k].numel()] = torch.fft.fft2(img, norm="ortho").reshape(nc, -1)[:, idx[k]]
    return y


def _adjoint(case, coils, idx, y):
    nc, ny, nx = case["nc"], case["ny"], case["nx"]
    X = torch.empty(case["q"], nx * ny, dtype=torch.complex128, device=DEV)
    for k in range(case["q"]):
        full = torch.zeros(nc, nx * ny, dtype=torch.complex128, device=DEV)
        full[:, idx[k]] = y[k, :, :idx[k].numel()]
        img = torch.fft.ifft2(full.reshape(nc, ny, nx), norm="ortho").reshape(nc, -1)
        X[k] = (coils.conj() * img).sum(0)
    return X


def _crandn(gen, *shape):
    return torch.complex(torch.randn(*shape, device=DEV, generator=gen, dtype=torch.float64),
                         torch.randn(*shape, device=DEV, generator=gen, dtype=torch.float64)) / math.sqrt(2.0)


def _orth(A):
    """Rows of A (r, n) made orthonormal: the Q factor with a positive diagonal R of A^T."""
    A = A.to(torch.complex128)
    for _ in range(2):
        G = (A.conj() @ A.T.contiguous()).cpu()  # r x r: <a_i, a_j>
        R = torch.linalg.cholesky(G).conj().T.contiguous()  # G = R^H R with G_ij = a_i^H a_j
        A = torch.linalg.inv(R).T.contiguous().to(A.device) @ A
    return A


def _basis(Z, r, noise, gen):
    """An orthonormal (r, n) complex64 basis near the sequence's leading subspace (on the host: the
    same bits from the same seed, whatever order a GPU's matrix product adds in)."""
    Zh = Z.cpu().numpy()
    w, V = np.linalg.eigh(Zh.conj() @ Zh.T)
    U = V[:, ::-1][:, :r].T @ Zh if r <= Zh.shape[0] else _crandn(gen, r, Zh.shape[1]).cpu().numpy()
    U = U / np.sqrt((np.abs(U) ** 2).sum(1, keepdims=True))
    U = U + noise / math.sqrt(Z.shape[1]) * _crandn(gen, *U.shape).cpu().numpy()
    for _ in range(2):
        R = np.linalg.cholesky(U.conj() @ U.T).conj().T
        U = np.linalg.inv(R).T @ U
    return torch.from_numpy(U.astype(np.complex64)).to(DEV)


def _inputs(case, seed):
    rng = np.random.default_rng([int(seed), 77])
    gen = torch.Generator(device=DEV).manual_seed(int(seed) + 1)
    nx, ny, q, r = case["nx"], case["ny"], case["q"], case["r"]
    n = nx * ny
    d = {}
    if case["op"] == "cnn":
        b = case["batch"]
        x, t = [], []
        for i in range(b):
            Z = _sequence(nx, ny, q, rng, gen)
            t.append(_basis(Z, r, 0.0, gen))  # the target: the sequence's own leading basis
            Z = Z + 0.1 * _crandn(gen, q, n)
            x.append(torch.view_as_real(Z).permute(0, 2, 1).reshape(2 * q, ny, nx))
        x = torch.stack(x)
        d["x"] = (x / x.square().mean((1, 2, 3), keepdim=True).sqrt()).to(torch.float32)
        d["Ut"] = torch.stack(t)
        p = []
        for ci, co in _layers(case):
            p.append(torch.randn(co * ci * 9, device=DEV, generator=gen, dtype=torch.float64) * math.sqrt(2.0 / (9 * ci)))
            p.append(0.02 * torch.randn(co, device=DEV, generator=gen, dtype=torch.float64))
        d["params"] = torch.cat(p).to(torch.float32)
        return d
    masks = _masks(case, rng)
    idx = _flat(case, masks)
    per = nx if case["mask"] == "lines" else 1
    m_k = [len(m) * per for m in masks]
    m_max, width = max(m_k), max(len(m) for m in masks)
    pad = -np.ones((q, width), dtype=np.int32)
    for k, m in enumerate(masks):
        pad[k, :len(m)] = m
    coils = _coil_maps(nx, ny, case["nc"])
    c128 = coils.to(torch.complex128)
    d.update(coils=coils, idx=idx, m_max=m_max, mask=torch.from_numpy(pad).to(DEV),
             m_k=torch.tensor(m_k, dtype=torch.int32, device=DEV))
    op = case["op"]
    if op in ("mec1", "mec2"):  # the error left by a low-rank fit: a sparse, structured part and noise
        Z = 0.1 * _crandn(gen, q, n) * (torch.rand(q, n, device=DEV, generator=gen) < 0.05)
        Z = Z + 0.02 * (_sequence(nx, ny, q, rng, gen) - _sequence(nx, ny, q, rng, gen))
    else:
        Z = _sequence(nx, ny, q, rng, gen)
    if op == "ops":
        d["X"] = Z.to(torch.complex64)
        return d
    y = _forward(case, c128, idx, Z, m_max)
    valid = (torch.arange(m_max, device=DEV)[None, :] < d["m_k"][:, None])[:, None, :]
    power = y.abs().square().sum() / (case["nc"] * sum(m_k))
    y = torch.where(valid, y + torch.sqrt(power * 1e-3) * _crandn(gen, *y.shape), torch.zeros_like(y))
    d["y"] = y.to(torch.complex64)
    if op == "steps":
        d["U0"] = _basis(Z, r, 0.1, gen)
    if op == "online":  # mean and basis of the frames before
        past = _sequence(nx, ny, 24, rng, gen)
        zbar = past.mean(0)
        d["zbar"] = zbar.to(torch.complex64)
        d["U0"] = _basis(past - zbar[None, :], r, 0.02, gen)
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    if case["op"] == "cnn":
        net = ag.WsInit(case["nx"], case["ny"], case["q"], case["r"], width=32, batch=case["batch"])
        return dict(case=case, net=net, **d)
    d.pop("idx")
    kind = ag.MASK_LINES if case["mask"] == "lines" else ag.MASK_INDEX
    ctx = ag.AltGDmin(case["nx"], case["ny"], case["nc"], case["q"], case["r"], d["m_max"], kind,
                      ag.MIXED if case["mixed"] else ag.FP32)
    ctx.set_problem(d["coils"], d["mask"], d["m_k"], d.get("y"))
    n = case["nx"] * case["ny"]
    s = dict(case=case, ctx=ctx, workspace=ctx._keep[4], **d)
    if case["op"] in ("recon", "steps", "init"):
        s["U"] = torch.empty(case["r"], n, dtype=torch.complex64, device=DEV)
        s["U_prev"] = torch.empty_like(s["U"])
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _bind(s, y):
    s["ctx"].set_problem(s["coils"], s["mask"], s["m_k"], y, workspace=s["workspace"])


def run(s):
    case, op = s["case"], s["case"]["op"]
    if op == "cnn":
        loss, grads = s["net"].loss_backward(s["params"], s["x"], s["Ut"])
        return {"loss": loss, "grads": grads}
    ctx = s["ctx"]
    if op == "recon":
        _bind(s, s["y"])
        U = ctx.init(s["U"])
        B = ctx.iterate(case["iters"], U, U_prev=s["U_prev"])
        return ctx.expand(s["U_prev"], B)
    if op == "steps":
        U = ctx.init_from(s["U0"], s["U"])
        B = ctx.iterate(case["iters"], U, U_prev=s["U_prev"])
        return {"U": U, "U_prev": s["U_prev"], "B": B}
    if op == "init":
        U = ctx.init(s["U"])
        return ctx.expand(U, ctx.ls(U))
    if op == "online":
        _bind(s, s["y"])
        yt = ctx.residual(zbar=s["zbar"])
        _bind(s, yt)
        b = ctx.ls(s["U0"])
        e = ctx.mec_cgls(ctx.residual(X=ctx.expand(s["U0"], b)), 3, 1e-36)
        return {"b": b, "e": e, "z": ctx.expand(s["U0"], b, s["zbar"], e)}
    if op == "mean":
        return ctx.mean(1e-3, 10)
    if op == "mec1":
        return ctx.mec_cgls(s["y"], 3, 1e-36)
    if op == "mec2":
        return ctx.mec_ista(s["y"], 10, 1e-3, 0.0025)
    Y = ctx.apply_A(s["X"])
    return {"Y": Y, "X": ctx.apply_AH(Y)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _layers(case):
    return [(2 * case["q"], 32), (32, 32), (32, 32), (32, 2 * case["r"])]


def work(case):
    nx, ny, nc, q, r = (case[k] for k in ("nx", "ny", "nc", "q", "r"))
    n = nx * ny
    if case["op"] == "cnn":
        par = sum(ci * co * 9 + co for ci, co in _layers(case))
        mac = sum(ci * co * 9 for ci, co in _layers(case)) * n * case["batch"]
        first = _layers(case)[0][0] * 32 * 9 * n * case["batch"]  # the images need no gradient
        return {"bytes": 4.0 * case["batch"] * n * 2 * q + 8.0 * case["batch"] * n * r + 8.0 * par,
                "flops": 2.0 * (3 * mac - first)}
    lines = case["mask"] == "lines"
    # samples per frame and coil, and k-space locations sampled by any frame
    m = case["lines"] * nx * (0.875 if case["ragged"] else 1.0) if lines else 0.7 * case["spokes"] * max(nx, ny)
    locs = min(float(n), m * q)
    M = m * q
    fft = (5.0 * n * math.log2(ny) if lines else 5.0 * n * math.log2(n)) + 8.0 * n  # one coil image, weighted
    it = 2.0 * nc * r * fft + 8.0 * nc * M * r * 2 + 8.0 * nc * r * r * ((locs if lines else M) + locs)
    op_fft = 5.0 * n * math.log2(n) + 8.0 * n
    b_in = 8.0 * nc * M + 8.0 * nc * n
    op = case["op"]
    if op == "recon":
        return {"bytes": b_in + 8.0 * n * q, "flops": case["iters"] * it + nc * q * op_fft + 4.0 * n * q * q + 8.0 * n * q * r * 2}
    if op == "steps":
        return {"bytes": b_in + 8.0 * n * r * 3, "flops": case["iters"] * it + 8.0 * n * r * r}
    if op == "init":
        return {"bytes": b_in + 8.0 * n * q, "flops": nc * q * op_fft + 4.0 * n * q * q + 8.0 * n * q * r * 2 + it}
    if op == "online":
        return {"bytes": b_in + 8.0 * n * (r + 3), "flops": nc * op_fft * 9 + nc * r * fft + 16.0 * n * r}
    if op == "mean":
        return {"bytes": b_in + 8.0 * n, "flops": nc * q * op_fft + 10 * 2 * nc * fft}
    if op == "mec1":
        return {"bytes": b_in + 8.0 * n * q, "flops": 7.0 * nc * q * op_fft}
    if op == "mec2":
        return {"bytes": b_in + 8.0 * n * q, "flops": 20.0 * nc * q * op_fft + 10 * 2 * 5.0 * n * q * math.log2(max(q, 2))}
    return {"bytes": 8.0 * nc * n + 2 * 8.0 * n * q + 8.0 * nc * M, "flops": 2.0 * nc * q * op_fft}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
class _Exact:
    """A_k U by shared coil-image transforms, the LS step and the gradient."""

    def __init__(self, case, d):
        self.case, self.idx, self.m_max = case, d["idx"], d["m_max"]
        self.coils = d["coils"].to(torch.complex128)
        self.y = d["y"].to(torch.complex128)

    def basis(self, U):
        """W (nc, n, r): the coil-weighted transforms of U (r, n)."""
        c = self.case
        img = (self.coils[:, None, :] * U[None, :, :]).reshape(c["nc"], U.shape[0], c["ny"], c["nx"])
        W = torch.fft.fft2(img, norm="ortho").reshape(c["nc"], U.shape[0], -1)
        return W.permute(0, 2, 1).contiguous()

    def ls(self, W, y):
        B, A = [], []
        r = W.shape[2]
        for k in range(self.case["q"]):
            a = W[:, self.idx[k], :].reshape(-1, r)
            yk = y[k, :, :self.idx[k].numel()].reshape(-1)
            ah = a.conj().T.contiguous()
            A.append((ah @ a, ah @ yk))
        G = torch.stack([g for g, _ in A]).cpu()
        h = torch.stack([v for _, v in A]).cpu()
        return torch.linalg.solve(G, h).to(DEV)  # (q, r)

    def gradient(self, U):
        c = self.case
        r, n = U.shape
        W = self.basis(U)
        B = self.ls(W, self.y)
        K = torch.zeros(c["nc"], n, r, dtype=torch.complex128, device=DEV)
        for k in range(c["q"]):
            i = self.idx[k]
            res = W[:, i, :] @ B[k] - self.y[k, :, :i.numel()]
            K.index_add_(1, i, res[:, :, None] * B[k].conj()[None, None, :])
        img = torch.fft.ifft2(K.permute(0, 2, 1).contiguous().reshape(c["nc"], r, c["ny"], c["nx"]), norm="ortho")
        G = (self.coils.conj()[:, None, :] * img.reshape(c["nc"], r, n)).sum(0)
        return B, G

    def loop(self, U, iters):
        eta, prev, B = None, U, None
        for _ in range(iters):
            B, G = self.gradient(U)
            if eta is None:
                s2 = torch.linalg.eigvalsh((G.conj() @ G.T.contiguous()).cpu())[-1]
                eta = 0.14 / math.sqrt(float(s2))
            prev, U = U, _orth(U - eta * G)
        return U, prev, B

    def init(self):
        c = self.case
        m_k = [i.numel() for i in self.idx]
        gamma = 36.0 * float(self.y.abs().square().sum()) / (max(m_k) * c["q"])
        yt = torch.where(self.y.abs().square() <= gamma, self.y, torch.zeros_like(self.y))
        X = _adjoint(c, self.coils, self.idx, yt)
        mbar = sum(m_k) / c["q"]
        X = X / torch.sqrt(torch.tensor(m_k, dtype=torch.float64, device=DEV) * mbar)[:, None]
        w, V = np.linalg.eigh((X.conj() @ X.T.contiguous()).cpu().numpy())
        V = torch.from_numpy(np.ascontiguousarray(V[:, ::-1][:, :c["r"]])).to(DEV)
        return _orth((X.T.contiguous() @ V).T.contiguous())


def _exact_cgls(case, coils, idx, y, iters):
    """Per frame: CGLS from zero on ||y_k - A_k e||."""
    m_max = y.shape[2]
    dot = lambda a: a.abs().square().reshape(a.shape[0], -1).sum(1)  # noqa: E731
    r, s = y.clone(), _adjoint(case, coils, idx, y)
    e, p, g = torch.zeros_like(s), s.clone(), dot(s)
    for _ in range(iters):
        w = _forward(case, coils, idx, p, m_max)
        a = g / dot(w)
        e, r = e + a[:, None] * p, r - a[:, None, None] * w
        s = _adjoint(case, coils, idx, r)
        g2 = dot(s)
        p, g = s + (g2 / g)[:, None] * p, g2
    return e


def _exact_mean(case, coils, idx, y):
    n = case["nx"] * case["ny"]
    cnt = torch.zeros(n, dtype=torch.float64, device=DEV)
    for i in idx:
        cnt[i] += 1.0
    nc, ny, nx = case["nc"], case["ny"], case["nx"]

    def normal(z):
        f = torch.fft.fft2((coils * z[None, :]).reshape(nc, ny, nx), norm="ortho") * cnt.reshape(1, ny, nx)
        return (coils.conj() * torch.fft.ifft2(f, norm="ortho").reshape(nc, n)).sum(0)

    s = _adjoint(case, coils, idx, y).sum(0)
    x, p, g = torch.zeros_like(s), s.clone(), float(s.abs().square().sum())
    g0 = g
    for _ in range(10):
        w = normal(p)
        a = g / float((p.conj() * w).sum().real)
        x, s = x + a * p, s - a * w
        g2 = float(s.abs().square().sum())
        if math.sqrt(g2) <= 1e-3 * math.sqrt(g0):
            break
        p, g = s + (g2 / g) * p, g2
    return x


def _exact_ista(case, coils, idx, y):
    E = torch.zeros(case["q"], case["nx"] * case["ny"], dtype=torch.complex128, device=DEV)
    prev = omega = None
    for t in range(10):
        V = E + _adjoint(case, coils, idx, y - _forward(case, coils, idx, E, y.shape[2]))
        M = torch.fft.fft(V, dim=0, norm="ortho")
        mag = M.abs()
        if t == 0:
            omega = 1e-3 * float(mag.max())
            stop = False
        else:
            stop = float((M - prev).norm() / prev.norm()) < 0.0025
        S = torch.where(mag > omega, M * (1.0 - omega / torch.clamp(mag, min=1e-300)), torch.zeros_like(M))
        E = torch.fft.ifft(S, dim=0, norm="ortho")
        prev = M
        if stop:
            break
    return E


def _exact_cnn(case, d):
    nx, ny, r = case["nx"], case["ny"], case["r"]
    params = d["params"].to(torch.float64).requires_grad_(True)
    grads = torch.zeros_like(params)
    total = 0.0
    for b in range(case["batch"]):
        h, o = d["x"][b].to(torch.float64), 0
        for l, (ci, co) in enumerate(_layers(case)):
            W = params[o:o + co * ci * 9].reshape(co, ci, 3, 3)
            bias = params[o + co * ci * 9:o + co * ci * 9 + co]
            o += co * ci * 9 + co
            hp = torch.nn.functional.pad(h, (1, 1, 1, 1))
            out = bias[:, None].expand(co, nx * ny)
            for i in range(3):
                for j in range(3):
                    out = out + W[:, :, i, j] @ hp[:, i:i + ny, j:j + nx].reshape(ci, nx * ny)
            h = (torch.relu(out) if l < 3 else out).reshape(co, ny, nx)
        h = h.reshape(r, 2, nx * ny)
        M = torch.complex(h[:, 0], h[:, 1])  # (r, n)
        Ut = d["Ut"][b].to(torch.complex128)
        G = (M.conj() @ M.T.contiguous()).cpu()
        C = (M.conj() @ Ut.T.contiguous()).cpu()
        loss = (r - (torch.linalg.inv(G) @ C @ C.conj().T.contiguous()).diagonal().sum().real) / case["batch"]
        grads += torch.autograd.grad(loss, params)[0]
        total += float(loss.detach())
    return {"loss": torch.tensor([total], dtype=torch.float64), "grads": grads}


def exact(case, seed):
    d = _inputs(case, seed)
    op = case["op"]
    if op == "cnn":
        return _exact_cnn(case, d)
    idx, coils = d["idx"], d["coils"].to(torch.complex128)
    if op == "ops":
        Y = _forward(case, coils, idx, d["X"].to(torch.complex128), d["m_max"])
        return {"Y": Y, "X": _adjoint(case, coils, idx, Y)}
    y = d["y"].to(torch.complex128)
    if op == "mean":
        return _exact_mean(case, coils, idx, y)
    if op == "mec1":
        return _exact_cgls(case, coils, idx, y, 3)
    if op == "mec2":
        return _exact_ista(case, coils, idx, y)
    ex = _Exact(case, d)
    if op == "recon":
        _, prev, B = ex.loop(ex.init(), case["iters"])
        return B @ prev
    if op == "steps":
        U, prev, B = ex.loop(_orth(d["U0"]), case["iters"])
        return {"U": U, "U_prev": prev, "B": B}
    if op == "init":
        U = ex.init()
        return ex.ls(ex.basis(U), ex.y) @ U
    zbar, U0 = d["zbar"].to(torch.complex128), d["U0"].to(torch.complex128)
    yt = y - _forward(case, coils, idx, zbar[None, :], d["m_max"])
    b = ex.ls(ex.basis(U0), yt)
    fit = b @ U0
    e = _exact_cgls(case, coils, idx, yt - _forward(case, coils, idx, fit, d["m_max"]), 3)
    return {"b": b, "e": e, "z": zbar[None, :] + fit + e}
