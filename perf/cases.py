"""The work this framework is used for, as cases a timing program can run.

Each case is a dict of plain values; ``prepare`` makes what a program has in hand before
the call (device-resident stacks, sensor descriptions, workspaces, handles), ``run`` is one
pass through the public entry points, ``work`` the bytes and operations that pass cannot do
without, ``exact`` the same result in 64 bits from plain torch.

Kinds:

* ``im``        an interaction matrix from a stack of Gaussian influence functions: SCAO
                calibration, repeated whenever the misregistration estimate moves
                (engines: central differences, telescoping sum, edge repair);
* ``modal``     the same for dense modal maps through a clocked, anamorphic LGS sensor;
* ``jacobian``  the IM with its four derivative planes;
* ``step``      one forward and backward pass of the differentiable IM;
* ``mcao``      every (WFS, DM) pair of a multi-sensor system, maps renewed, graph replayed;
* ``warp``      the unfused steps: warp a stack, then its slopes;
* ``fit``       misregistration from measured probe slopes by Gauss-Newton;
* ``train``     one optimiser step of the learned estimator;
* ``proj``      the tomographic projection.
"""
import functools
import math

import numpy as np
import torch

import paper_2606_07759_amd as synim
from paper_2606_07759_amd import autograd, learned

DEV = "cuda"
COUPLING = 1.0 / math.sqrt(2.0 * math.log(1.0 / 0.15))   # Gaussian width per pitch, 15% coupling


# ------------------------------------------------------------------------------- cases
def listed():
    return [
        # online tracking on a small sensor: latency and launches are everything
        dict(name="scao8_im", kind="im", n_sub=8, p=10, grid=96, obscuration=0.0, engine="plain"),
        # the ELT-scale calibration, 5257 IFs of 512^2
        dict(name="elt_im", kind="im", n_sub=80, p=6, grid=512, obscuration=0.28,
             engine="plain"),
        # pre-masked IFs on a grid whose rows are no multiple of 16 bytes
        dict(name="repaired_im", kind="im", n_sub=37, p=7, grid=293, obscuration=0.28,
             engine="repaired"),
        # 4519 modes on an LGS sensor clocked by 15 degrees
        dict(name="modal_im", kind="modal", n_sub=68, p=7, grid=512, modes=4519, clock_deg=15.0,
             mag_y=0.97),
        # derivative planes for a tracking loop on an 8-m-class sensor
        dict(name="jacobian", kind="jacobian", n_sub=40, p=6, grid=272, obscuration=0.14),
        # one gradient step on theta, small sensor
        dict(name="gradient_step", kind="step", n_sub=8, p=10, grid=96, obscuration=0.0),
        # 6 LGS sensors x 3 DMs, 49 026 columns
        dict(name="mcao", kind="mcao", n_sub=68, p=7, grid=512, n_wfs=6, n_dm=3, n1d=81),
        # the two unfused steps on a slice of the ELT stack
        dict(name="warp_slopes", kind="warp", n_sub=80, p=6, grid=512, obscuration=0.28, n=1200),
        # tracking: one measurement at a time
        dict(name="fit_one", kind="fit", batch=1),
        # a campaign of measurements at once
        dict(name="fit_1000", kind="fit", batch=1000),
        # the estimator's training step at its own batch size
        dict(name="train_256", kind="train", batch=256),
        # tomographic projection of the MCAO system, 9 directions, pupil binned 4 x 4
        dict(name="projection", kind="proj", pupil=476, bin=4, grid=512, n_dm=3, n_layer=3,
             n_dir=9, pitch=6.0, layer_pitch=12.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid_for(rng, n_out):
    """An IF grid that holds the misregistered pupil: usually whole 16-byte rows, sometimes not."""
    g = n_out + 16 + n_out // 15
    return g + rng.randint(0, 7) if rng.random() < 0.3 else (g + 3) // 4 * 4


def draw(rng):
    kind = rng.choice(["im", "im", "im", "modal", "jacobian", "step", "mcao", "warp", "fit",
                       "fit", "train", "proj"])
    p = rng.randint(5, 10)
    if kind == "im":
        n_sub = _log_int(rng, 8, min(80, 480 // p))
        return dict(kind=kind, n_sub=n_sub, p=p, grid=_grid_for(rng, n_sub * p),
                    obscuration=rng.choice([0.0, 0.14, 0.28]),
                    engine=rng.choice(["plain", "plain", "tsum", "repaired"]))
    if kind == "modal":
        n_sub = _log_int(rng, 16, min(68, 476 // p))
        return dict(kind=kind, n_sub=n_sub, p=p, grid=(n_sub * p + 36 + 3) // 4 * 4,
                    modes=_log_int(rng, 200, 4000), clock_deg=round(rng.uniform(0.0, 20.0), 2),
                    mag_y=round(rng.uniform(0.96, 1.0), 3))
    if kind in ("jacobian", "step"):
        n_sub = _log_int(rng, 8, 40)
        p = rng.randint(5, 8)
        return dict(kind=kind, n_sub=n_sub, p=p, grid=_grid_for(rng, n_sub * p),
                    obscuration=rng.choice([0.0, 0.14, 0.28]))
    if kind == "mcao":
        n_sub = _log_int(rng, 20, 60)
        return dict(kind=kind, n_sub=n_sub, p=7, grid=(n_sub * 7 + 36 + 3) // 4 * 4,
                    n_wfs=rng.randint(2, 6), n_dm=rng.randint(1, 3), n1d=n_sub + 1)
    if kind == "warp":
        n_sub = _log_int(rng, 8, min(80, 480 // p))
        return dict(kind=kind, n_sub=n_sub, p=p, grid=_grid_for(rng, n_sub * p),
                    obscuration=rng.choice([0.0, 0.28]), n=_log_int(rng, 40, 1200))
    if kind == "fit":
        return dict(kind=kind, batch=_log_int(rng, 1, 1000))
    if kind == "train":
        return dict(kind=kind, batch=_log_int(rng, 32, 1000))
    return dict(kind="proj", pupil=4 * _log_int(rng, 25, 80), bin=rng.choice([2, 4]), grid=384,
                n_dm=rng.randint(1, 3), n_layer=rng.randint(1, 3), n_dir=rng.choice([1, 4, 9]),
                pitch=round(rng.uniform(8.0, 16.0), 2),
                layer_pitch=round(rng.uniform(14.0, 24.0), 2))


# ------------------------------------------------------------------------------ inputs
def _pupil(n, obscuration, offset=(0.0, 0.0)):
    c = (n - 1) / 2.0
    y, x = np.mgrid[0:n, 0:n].astype(np.float64)
    r = np.hypot(x - c - offset[0], y - c - offset[1])
    return ((r <= n / 2.0) & (r >= obscuration * n / 2.0)).astype(np.uint8)


def _valid(pupil, p):
    n = pupil.shape[0] // p
    frac = pupil.reshape(n, p, n, p).sum(axis=(1, 3)) / float(p * p)
    return np.flatnonzero(frac.ravel() >= 0.5).astype(np.int32)


def _actuators(n1d, pitch, grid, radius):
    c = (grid - 1) / 2.0
    pos = c + pitch * (np.arange(n1d) - (n1d - 1) / 2.0)
    x, y = np.meshgrid(pos, pos)
    keep = np.hypot(x - c, y - c) <= radius + pitch
    return x[keep], y[keep]


def _gauss_stack(n1d, pitch, grid, radius, rng, n=None):
    """float32 [n][grid][grid] Gaussian IFs, amplitudes N(1, 0.02) from ``rng``."""
    x, y = _actuators(n1d, pitch, grid, radius)
    if n is not None:
        pick = np.linspace(0, len(x) - 1, n).astype(int)
        x, y = x[pick], y[pick]
    amp = torch.from_numpy(rng.normal(1.0, 0.02, size=len(x))).to(DEV)
    t = torch.arange(grid, dtype=torch.float64, device=DEV)
    s2 = 2.0 * (COUPLING * pitch) ** 2
    gx = torch.exp(-(t[None] - torch.from_numpy(x).to(DEV)[:, None]) ** 2 / s2).float()
    gy = (amp[:, None] * torch.exp(-(t[None] - torch.from_numpy(y).to(DEV)[:, None]) ** 2 / s2)).float()
    out = torch.empty((len(x), grid, grid), dtype=torch.float32, device=DEV)
    torch.mul(gy[:, :, None], gx[:, None, :], out=out)
    return out


def _rng(seed):
    return np.random.Generator(np.random.PCG64(int(seed)))


def _theta(rng):
    """Shift within a pixel, rotation within a degree, magnification within 2%."""
    return (float(rng.uniform(-1, 1)), float(rng.uniform(-1, 1)),
            math.radians(float(rng.uniform(-1, 1))), float(rng.uniform(0.98, 1.02)))


def _dm_mask(case):
    """DM-side annulus the IFs of an edge-repaired build were multiplied by: 4 px inside the
    pupil's outer edge, 4 px outside its obscuration."""
    n, g = case["n_sub"] * case["p"], case["grid"]
    c = (g - 1) / 2.0
    y, x = np.mgrid[0:g, 0:g].astype(np.float64)
    r = np.hypot(x - c, y - c)
    return ((r <= n / 2.0 - 4) & (r >= (case["obscuration"] * n / 2.0 + 4 if case["obscuration"] else 0.0))).astype(np.uint8)


def _scao(case, seed):
    """(stack, theta, pupil, valid) of an SCAO case."""
    rng = _rng(seed)
    n = case["n_sub"] * case["p"]
    pupil = _pupil(n, case["obscuration"])
    theta = _theta(rng)
    F = _gauss_stack(case["n_sub"] + 1, float(case["p"]), case["grid"], n / 2.0, rng, case.get("n"))
    if case.get("engine") == "repaired":
        F *= torch.from_numpy(_dm_mask(case)).to(DEV).float()
    return F, theta, pupil, _valid(pupil, case["p"])


def _modal(case, seed):
    """(stack, composite geometry, pupil, valid): Fourier modes by spatial frequency, their
    amplitudes from the seed, an LGS sensor clocked and stretched behind a 4-km DM."""
    rng = _rng(seed)
    n, grid = case["n_sub"] * case["p"], case["grid"]
    r = int(math.ceil(math.sqrt(case["modes"] / math.pi))) + 2
    ks = [(kx, ky) for ky in range(r + 1) for kx in range(-r, r + 1) if (ky > 0 or kx > 0)]
    ks = sorted(ks, key=lambda k: (k[0] ** 2 + k[1] ** 2, math.atan2(k[1], k[0])))
    ks = np.repeat(np.array(ks, dtype=np.float64), 2, axis=0)[: case["modes"]]
    amp = rng.normal(1.0, 0.02, size=len(ks))
    t = (torch.arange(grid, dtype=torch.float64, device=DEV) - (grid - 1) / 2.0) * (2 * math.pi / n)
    F = torch.empty((len(ks), grid, grid), dtype=torch.float32, device=DEV)
    kx, ky, am = (torch.from_numpy(np.ascontiguousarray(v)).to(DEV) for v in (ks[:, 0], ks[:, 1], amp))
    for a in range(0, len(ks), 512):
        b = slice(a, min(len(ks), a + 512))
        ph = (kx[b, None, None] * t[None, None, :] + ky[b, None, None] * t[None, :, None]).float()
        F[b][0::2] = torch.cos(ph[0::2]) * am[b][0::2, None, None].float()
        F[b][1::2] = torch.sin(ph[1::2]) * am[b][1::2, None, None].float()
    cone = 1.0 - 4e3 / 90e3
    foot = 4e3 * math.radians(45 / 3600.0) / (39.0 / 476)
    g = dict(dm_shift_x=float(rng.uniform(-1, 1)), dm_shift_y=float(rng.uniform(-1, 1)),
             dm_rot=math.radians(0.3), dm_mag=1.003, cone_scale=cone,
             footprint_x=0.25 * foot, footprint_y=0.43 * foot, wfs_shift_x=0.4, wfs_shift_y=-0.7,
             wfs_rot=math.radians(case["clock_deg"]), wfs_mag_x=1.0, wfs_mag_y=case["mag_y"],
             kappa=1.0)
    pupil = _pupil(n, 0.28)
    return F, g, pupil, _valid(pupil, case["p"])


def _mcao(case, seed):
    """(stacks, wfs [(pupil, valid)], pairs [(wfs, dm, geometry)]): the sensors' clocking and
    pupil offsets belong to the case, the IF amplitudes and a small drift of each map to the seed."""
    rng = _rng(seed)
    fixed = _rng(7)
    n, p, grid = case["n_sub"] * case["p"], case["p"], case["grid"]
    H, alpha, pix = 90e3, math.radians(45 / 3600.0), 39.0 / n
    alts, scale = (0.0, 4e3, 12.7e3), (1.0, 80 / 46, 80 / 36)
    stacks, wfs, geo = [], [], []
    for d in range(case["n_dm"]):
        pitch = (n + 4.0) / (case["n1d"] - 1) * scale[d]
        n1d = int(round((n + 4.0) / pitch)) + 1
        stacks.append(_gauss_stack(n1d, pitch, grid, (n + 4) / 2.0, rng))
    for w in range(case["n_wfs"]):
        off = tuple(float(v) for v in fixed.uniform(-p / 2, p / 2, size=2))
        pupil = _pupil(n, 0.28, off)
        wfs.append((pupil, _valid(pupil, p)))
        az = math.radians(60.0 * w)
        rot = math.radians(math.degrees(az) % 90.0 - 45.0)
        for d in range(case["n_dm"]):
            f = alts[d] * alpha / pix
            geo.append((w, d, dict(
                dm_shift_x=float(rng.uniform(-0.2, 0.2)), dm_shift_y=float(rng.uniform(-0.2, 0.2)),
                dm_rot=0.0, dm_mag=1.0, cone_scale=1.0 - alts[d] / H,
                footprint_x=f * math.cos(az), footprint_y=f * math.sin(az), wfs_shift_x=off[0],
                wfs_shift_y=off[1], wfs_rot=rot, wfs_mag_x=1.0, wfs_mag_y=1.0, kappa=1.0)))
    return stacks, wfs, geo


@functools.lru_cache(maxsize=1)
def _probe_system():
    return learned.probe_system(DEV)


def _probe_fit(case, seed):
    """(measured slopes [B][M] float32, the sensor's pupil and valid list, probes)."""
    s = _probe_system()
    g = torch.Generator(device="cpu").manual_seed(int(seed))
    B = case["batch"]
    lo, hi = torch.from_numpy(s.lo), torch.from_numpy(s.hi)
    th = lo + torch.rand((B, 4), generator=g, dtype=torch.float64) * (hi - lo)
    snr = 20.0 + 180.0 * torch.rand(B, generator=g, dtype=torch.float64)
    noise = torch.randn((B, s.M), generator=g, dtype=torch.float64)
    S = _probe_slopes64(s, th.to(DEV))[0]
    rms = S.square().mean(dim=1, keepdim=True).sqrt()
    return (S + noise.to(DEV) * rms / snr.to(DEV)[:, None]).float().contiguous(), s


def _train_state(case, seed):
    """A network in mid-training with one batch: parameters, Adam moments, inputs, targets."""
    s = _probe_system()
    net = learned.net_for(s)
    B = case["batch"]
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    d = net.desc
    parts = []
    for o, i in ((d.h1, d.n_in), (d.h2, d.h1), (d.n_out, d.h2)):
        parts += [torch.randn(o * i, generator=g, device=DEV) * math.sqrt(2.0 / i),
                  torch.randn(o, generator=g, device=DEV) * 0.01]
    params = torch.cat(parts)
    x = torch.randn((B, s.M), generator=g, device=DEV)
    t = torch.rand((B, 4), generator=g, device=DEV) * 2 - 1
    v = (torch.rand(params.numel(), generator=g, device=DEV) + 0.1) * 1e-5
    m = torch.randn(params.numel(), generator=g, device=DEV) * 1e-3
    return net, params, m, v, x, t


def _proj_inputs(case, seed):
    rng = _rng(seed)
    n, grid = case["pupil"], case["grid"]
    pix = 39.0 / 476
    R = n / 2.0 + 2.0
    comps = []
    for alts, scales, count, pitch in (((0.0, 4e3, 12.7e3), (1.0, 80 / 46, 80 / 36), case["n_dm"], case["pitch"]),
                                       ((2e3, 8e3, 16e3), (1.0, 1.0, 1.0), case["n_layer"], case["layer_pitch"])):
        comps.append([(_gauss_stack(int(round(2 * R / (pitch * s))) + 1, pitch * s, grid, R, rng), h, pix)
                      for h, s in zip(alts[:count], scales[:count])])
    a = math.radians(40 / 3600.0)
    dirs = np.array([[x * a, y * a] for y in (-1, 0, 1) for x in (-1, 0, 1)])
    pick = {1: [4], 4: [0, 2, 6, 8], 9: list(range(9))}[case["n_dir"]]
    # a thousandth of the diagonal a unit Gaussian of this pitch has in the Gram matrix
    lam = 1e-3 * case["n_dir"] * math.pi * (COUPLING * case["pitch"] / case["bin"]) ** 2
    return comps[0], comps[1], dirs[pick], _pupil(n, 0.28), pix, lam


# ----------------------------------------------------------------------------- prepare
class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    kind = case["kind"]
    if kind in ("im", "jacobian", "step", "warp"):
        s.F, s.theta, pupil, valid = _scao(case, seed)
        s.wfs = synim.Wfs.from_numpy(pupil, case["p"], valid, device=DEV)
        H, W = s.wfs.shape
        s.A, s.dA = synim.affine_from_misreg(s.theta, case["grid"], case["grid"], H, W)
        n = s.F.shape[0]
        if kind in ("im", "warp"):
            s.out = torch.empty((n, 2 * s.wfs.n_valid), dtype=torch.float32, device=DEV)
        if kind == "im" and case["engine"] == "repaired":
            s.mask = torch.from_numpy(_dm_mask(case)).to(DEV)
        elif kind in ("im", "jacobian"):
            planes = 1 if kind == "im" else 5
            s.ws = torch.empty(synim.im_workspace_bytes(s.wfs, s.A, planes), dtype=torch.uint8, device=DEV)
        if kind == "warp":
            s.phase = torch.empty((n, H + 2, W + 2), dtype=torch.float32, device=DEV)
        if kind == "step":
            g = torch.Generator(device=DEV).manual_seed(int(seed))
            s.t = torch.tensor(s.theta, dtype=torch.float64, requires_grad=True)
            s.grad = torch.randn((n, 2 * s.wfs.n_valid), generator=g, device=DEV)
    elif kind == "modal":
        s.F, g, pupil, valid = _modal(case, seed)
        s.wfs = synim.Wfs.from_numpy(pupil, case["p"], valid, device=DEV)
        H, W = s.wfs.shape
        s.A = synim.affine_from_geometry(_Geometry(g), case["grid"], case["grid"], H, W)
        s.ws = torch.empty(synim.im_workspace_bytes(s.wfs, s.A, 1), dtype=torch.uint8, device=DEV)
        s.out = torch.empty((s.F.shape[0], 2 * s.wfs.n_valid), dtype=torch.float32, device=DEV)
    elif kind == "mcao":
        stacks, wfs, geo = _mcao(case, seed)
        n_out = case["n_sub"] * case["p"]
        w = [synim.Wfs.from_numpy(P, case["p"], v, device=DEV) for P, v in wfs]
        s.maps = [synim.affine_from_geometry(_Geometry(g), case["grid"], case["grid"], n_out, n_out)
                  for _, _, g in geo]
        s.batch = synim.Batch(w, stacks, [(a, b, A) for (a, b, _), A in zip(geo, s.maps)], device=DEV)
    elif kind == "fit":
        s.slopes, sys_ = _probe_fit(case, seed)
        s.ctx = synim.Misreg(sys_.wfs, sys_.probes, sys_.lo, sys_.hi, max_batch=case["batch"])
        s.out = (torch.empty((case["batch"], 4), dtype=torch.float64, device=DEV),
                 torch.empty(case["batch"], dtype=torch.int32, device=DEV))
    elif kind == "train":
        s.net, s.params, s.m, s.v, s.x, s.t = _train_state(case, seed)
        s.grads = torch.empty_like(s.params)
        s.scratch = s.net.scratch(case["batch"], device=DEV)
        s.y = torch.empty((case["batch"], 4), dtype=torch.float32, device=DEV)
        s.loss = torch.empty(1, dtype=torch.float32, device=DEV)
        s.step = 1000
    else:
        s.args = _proj_inputs(case, seed)
        dms, layers, dirs, pupil, _, _ = s.args
        s.ws = torch.empty(synim.proj_workspace_bytes(dms, layers, len(dirs), pupil, case["bin"]),
                           dtype=torch.uint8, device=DEV)
    return s


class _Geometry:
    def __init__(self, fields):
        self.__dict__.update(fields)


# --------------------------------------------------------------------------------- run
def run(s):
    kind = s.case["kind"]
    if kind == "modal" or (kind == "im" and s.case["engine"] == "plain"):
        return synim.im_build(s.F, s.A, s.wfs, out=s.out, ws=s.ws)
    if kind == "im":
        if s.case["engine"] == "tsum":
            return synim.im_build_tsum(s.F, s.A, s.wfs, out=s.out, ws=s.ws)
        return synim.im_build_repaired(s.F, s.mask, s.A, s.wfs, out=s.out)
    if kind == "jacobian":
        return synim.im_jacobian(s.F, s.A, s.dA, s.wfs, ws=s.ws)
    if kind == "step":
        s.t.grad = None
        im = autograd.interaction_matrix(s.t, s.F, s.wfs)
        im.backward(s.grad)
        return im.detach(), s.t.grad
    if kind == "mcao":
        s.batch.set_maps(s.maps)
        return s.batch.run_graph()
    if kind == "warp":
        H, W = s.wfs.shape
        synim.affine_warp(s.F, s.A, H, W, halo=1, out=s.phase)
        return s.phase, synim.sa_slopes(s.phase, s.wfs, out=s.out)
    if kind == "fit":
        return s.ctx.infer(s.slopes, synim.MISREG_GN, out=s.out)
    if kind == "train":
        s.net.forward(s.params, s.x, s.scratch, s.y)
        s.net.backward(s.params, s.x, s.scratch, s.y, s.t, s.grads, s.loss)
        s.step += 1
        synim.adam_step(s.params, s.grads, s.m, s.v, s.step, lr=1e-4)
        return s.y, s.loss, s.grads, s.params, s.m, s.v
    dms, layers, dirs, pupil, pix, lam = s.args
    return synim.proj_opt(dms, layers, dirs, pupil, pix, lam, bin=s.case["bin"], ws=s.ws)


# -------------------------------------------------------------------------------- work
def _samples(pupil):
    """Haloed samples that central differences over the pupil read."""
    q = np.zeros((pupil.shape[0] + 2, pupil.shape[1] + 2), bool)
    u = pupil > 0
    q[1:-1, 2:] |= u
    q[1:-1, :-2] |= u
    q[2:, 1:-1] |= u
    q[:-2, 1:-1] |= u
    return int(q.sum())


def _annulus(n, obscuration):
    return math.pi / 4 * n * n * (1 - obscuration ** 2)


def _n_act(n1d, pitch, grid, radius):
    return len(_actuators(n1d, pitch, grid, radius)[0])


def work(case):
    """Bytes: each influence function's pixels under the pupil once, each result once.  Operations:
    a bilinear sample (8) per point the slopes read, its difference and sum."""
    kind = case["kind"]
    if kind in ("im", "jacobian", "step", "warp", "modal"):
        n = case["n_sub"] * case["p"]
        ob = case.get("obscuration", 0.28)
        pupil = _pupil(n, ob)
        nv, pts = len(_valid(pupil, case["p"])), _samples(pupil)
        na = case["modes"] if kind == "modal" else case.get("n") or _n_act(
            case["n_sub"] + 1, float(case["p"]), case["grid"], n / 2.0)
        if kind == "warp":
            win = (n + 2) ** 2
            return {"bytes": na * (4.0 * n * n + 4.0 * win + 8 * nv), "flops": na * (8.0 * win + 6.0 * n * n)}
        planes = {"jacobian": 5, "step": 1}.get(kind, 1)
        # the gradient step reads the stack for the forward and again for the backward pass
        reads = 2 if kind == "step" else 1
        by = na * (reads * 4.0 * _annulus(n, ob) + 8.0 * nv * (planes + (1 if kind == "step" else 0)))
        return {"bytes": by, "flops": na * pts * (12.0 if planes == 1 and kind != "step" else 44.0)}
    if kind == "mcao":
        n = case["n_sub"] * case["p"]
        by = fl = 0.0
        scale = (1.0, 80 / 46, 80 / 36)
        pupil = _pupil(n, 0.28)
        nv, pts = len(_valid(pupil, case["p"])), _samples(pupil)
        for d in range(case["n_dm"]):
            pitch = (n + 4.0) / (case["n1d"] - 1) * scale[d]
            na = _n_act(int(round((n + 4.0) / pitch)) + 1, pitch, case["grid"], (n + 4) / 2.0)
            by += na * (4.0 * math.pi / 4 * n * n + 8.0 * nv * case["n_wfs"])
            fl += na * 12.0 * pts * case["n_wfs"]
        return {"bytes": by, "flops": fl}
    if kind == "fit":
        # six Gauss-Newton steps of 20 probes on 52 subapertures, about 64 points each, value and
        # gradient of a bilinear sample with its moments (60)
        return {"bytes": case["batch"] * (2080 * 4 + 36.0) + 20 * 128 * 128 * 4.0,
                "flops": case["batch"] * 6 * 20 * 52 * 64 * 60.0}
    if kind == "train":
        B, K, h1, h2 = case["batch"], 2080, 512, 256
        P = 8000 * h1 + h1 + h2 * h1 + h2 + 4 * h2 + 4
        # parameters and both moments read and written once, the gradient written once
        return {"bytes": 4.0 * (7 * P + B * K), "flops": 2.0 * B * (2 * K * h1 + 3 * h1 * h2 + 12 * h2) + 12.0 * P}
    n, R = case["pupil"], case["pupil"] / 2.0 + 2.0
    scale = (1.0, 80 / 46, 80 / 36)
    nd = sum(_n_act(int(round(2 * R / (case["pitch"] * s))) + 1, case["pitch"] * s, case["grid"], R)
             for s in scale[: case["n_dm"]])
    nl = case["n_layer"] * _n_act(int(round(2 * R / case["layer_pitch"])) + 1, case["layer_pitch"], case["grid"], R)
    rows = _blocks(_pupil(n, 0.28), case["bin"])[0].size * case["n_dir"]
    return {"bytes": 4.0 * (nd + nl) * math.pi / 4 * n * n + 8.0 * nd * nl,
            "flops": float(rows) * nd * nd + 2.0 * rows * nd * nl + nd ** 3 / 3.0 + 2.0 * nd * nd * nl}


# ------------------------------------------------------------------------------- exact
def _inverse(theta, grid, n_out):
    """(A [2][2], b [2], dA [4] of [2][3]) of p_s = A p_o + b for a misregistration."""
    tx, ty, rot, m = theta
    c, s = math.cos(rot) / m, math.sin(rot) / m
    A = np.array([[c, s], [-s, c]])
    cs, co = (grid - 1) / 2.0, np.array([(n_out - 1) / 2.0 + tx, (n_out - 1) / 2.0 + ty])
    dR = np.array([[-s, c], [-c, -s]])
    planes = [np.column_stack([np.zeros((2, 2)), -A[:, 0]]), np.column_stack([np.zeros((2, 2)), -A[:, 1]]),
              np.column_stack([dR, -dR @ co]), np.column_stack([-A / m, A @ co / m])]
    return A, cs - A @ co, planes


def _inverse_geometry(g, grid, n_out):
    def rot(a):
        return np.array([[math.cos(a), -math.sin(a)], [math.sin(a), math.cos(a)]])
    W = np.diag([g["wfs_mag_x"], g["wfs_mag_y"]]) @ rot(g["wfs_rot"])
    L = W / (g["kappa"] * g["cone_scale"])
    M = L @ (g["dm_mag"] * rot(g["dm_rot"]))
    t = L @ (np.array([g["dm_shift_x"], g["dm_shift_y"]]) - np.array([g["footprint_x"], g["footprint_y"]]))
    t = t + np.array([g["wfs_shift_x"], g["wfs_shift_y"]])
    A = np.linalg.inv(M)
    return A, (grid - 1) / 2.0 - A @ ((n_out - 1) / 2.0 + t)


def _taps(xs, ys, H, W):
    """[(flat index, weight)] of the four bilinear taps, outside ones weighted zero, and the
    weights' derivatives along x and y."""
    i, j = torch.floor(xs), torch.floor(ys)
    a, c = xs - i, ys - j
    out = []
    for di, dj, w, wx, wy in ((0, 0, (1 - a) * (1 - c), c - 1, a - 1), (1, 0, a * (1 - c), 1 - c, -a),
                              (0, 1, (1 - a) * c, -c, 1 - a), (1, 1, a * c, c, a)):
        x, y = i + di, j + dj
        ok = ((x >= 0) & (x < W) & (y >= 0) & (y < H)).double()
        idx = (y.clamp(0, H - 1) * W + x.clamp(0, W - 1)).long()
        out.append((idx, w * ok, wx * ok, wy * ok))
    return out


def _gather(F, taps, k=1):
    flat = F.reshape(F.shape[0], -1)
    out = 0.0
    for t in taps:
        out = out + flat[:, t[0].reshape(-1)].double() * t[k].reshape(1, -1)
    return out.reshape(F.shape[0], *taps[0][0].shape)


def _points(A, b, x, y):
    return A[0, 0] * x + A[0, 1] * y + b[0], A[1, 0] * x + A[1, 1] * y + b[1]


def _window(n_out):
    t = torch.arange(-1, n_out + 1, dtype=torch.float64, device=DEV)
    return t[None, :].expand(n_out + 2, -1), t[:, None].expand(-1, n_out + 2)


def _sub_means(gx, gy, pupil, p, valid):
    """[n][2N] means of pupil-masked pixel values over the valid subapertures."""
    P = torch.from_numpy(pupil).to(DEV).double()
    ns = pupil.shape[0] // p
    v = torch.from_numpy(valid).to(DEV).long()
    nk = P.reshape(ns, p, ns, p).sum((1, 3)).reshape(-1)[v]
    return torch.cat([(g * P).reshape(-1, ns, p, ns, p).sum((2, 4)).reshape(-1, ns * ns)[:, v] / nk
                      for g in (gx, gy)], dim=1)


def _differences(phi, pupil, p, valid):
    gx = (phi[:, 1:-1, 2:] - phi[:, 1:-1, :-2]) / 2
    gy = (phi[:, 2:, 1:-1] - phi[:, :-2, 1:-1]) / 2
    return _sub_means(gx, gy, pupil, p, valid)


def _repair(phi, mask, A, b, n_out):
    x, y = _window(n_out)
    g = mask.shape[0]
    core = _gather(mask[None], _taps(*_points(A, b, x, y), g, g))[0] >= 0.999999
    pad = torch.nn.functional.pad(core.double(), (2, 2, 2, 2))
    h = n_out + 2

    def at(t, dx, dy):
        return t[..., 2 + dy:2 + dy + h, 2 + dx:2 + dx + h]
    ph = torch.nn.functional.pad(phi * core, (2, 2, 2, 2))
    total, count = 0.0, 0.0
    for dx, dy in ((1, 0), (-1, 0), (0, 1), (0, -1)):
        s1, s2 = at(pad, dx, dy), at(pad, 2 * dx, 2 * dy)
        p1, p2 = at(ph, dx, dy), at(ph, 2 * dx, 2 * dy)
        total = total + s1 * (p1 + s2 * (p1 - p2))
        count = count + s1
    ring = (~core & (count > 0)).double()
    return phi * core + ring * total / count.clamp(min=1)


def _chunks(n, cells):
    step = max(1, int(2e8 // cells))
    return [slice(a, min(n, a + step)) for a in range(0, n, step)]


def _build64(F, A, b, pupil, p, valid, planes=None, engine="plain", mask=None):
    """The IM in 64 bits (and with ``planes`` its derivative planes [4][n][2N])."""
    n_out, g = pupil.shape[0], F.shape[1]
    x, y = _window(n_out)
    taps = _taps(*_points(A, b, x, y), g, g)
    im, dim = [], [[] for _ in planes or ()]
    for c in _chunks(F.shape[0], 5 * (n_out + 2) ** 2):
        if engine == "tsum":
            t = torch.arange(n_out, dtype=torch.float64, device=DEV)
            e = torch.arange(n_out + 1, dtype=torch.float64, device=DEV) - 0.5
            hx = _gather(F[c], _taps(*_points(A, b, e[None, :].expand(n_out, -1), t[:, None].expand(-1, n_out + 1)), g, g))
            hy = _gather(F[c], _taps(*_points(A, b, t[None, :].expand(n_out + 1, -1), e[:, None].expand(-1, n_out)), g, g))
            im.append(_sub_means(hx[:, :, 1:] - hx[:, :, :-1], hy[:, 1:] - hy[:, :-1], pupil, p, valid))
            continue
        phi = _gather(F[c], taps)
        if engine == "repaired":
            phi = _repair(phi, mask, A, b, n_out)
        im.append(_differences(phi, pupil, p, valid))
        if planes is not None:
            fx, fy = _gather(F[c], taps, 2), _gather(F[c], taps, 3)
            for j, d in enumerate(planes):
                dx, dy = _points(d[:, :2], d[:, 2], x, y)
                dim[j].append(_differences(fx * dx + fy * dy, pupil, p, valid))
    im = torch.cat(im)
    return im if planes is None else (im, torch.stack([torch.cat(d) for d in dim]))


def _probe_slopes64(s, theta, jac=False):
    """Probe slopes [B][M] (and their Jacobian [B][4][M]) at theta [B][4], in 64 bits: probe-major,
    x block then y block of each probe."""
    pupil, valid = s.wfs.pupil.cpu().numpy(), s.wfs.valid.cpu().numpy()
    n_out, g, p = pupil.shape[0], s.probes.shape[1], s.wfs.p
    x, y = _window(n_out)
    flat = s.probes.reshape(s.probes.shape[0], -1).double()
    S, J = [], []
    for th in theta.split(32 if jac else 128):
        tx, ty, rot, m = (th[:, k, None, None] for k in range(4))
        c, sn = torch.cos(rot) / m, torch.sin(rot) / m
        co = (n_out - 1) / 2.0
        u, v = x[None] - co - tx, y[None] - co - ty
        xs, ys = (g - 1) / 2.0 + c * u + sn * v, (g - 1) / 2.0 - sn * u + c * v
        taps = _taps(xs, ys, g, g)

        def field(k):
            out = 0.0
            for t in taps:
                out = out + flat[:, t[0].reshape(-1)].reshape(-1, *xs.shape) * t[k][None]
            return out.transpose(0, 1).reshape(-1, n_out + 2, n_out + 2)

        def slopes(phi):
            return _differences(phi, pupil, p, valid).reshape(len(th), -1)
        S.append(slopes(field(1)))
        if jac:
            fx, fy = field(2), field(3)
            n_p = flat.shape[0]
            dirs = ((-c, sn), (-sn, -c), (-sn * u + c * v, -c * u - sn * v),
                    (-(c * u + sn * v) / m, -(-sn * u + c * v) / m))
            J.append(torch.stack([slopes(fx * dx.expand_as(xs).repeat_interleave(n_p, 0) +
                                         fy * dy.expand_as(xs).repeat_interleave(n_p, 0))
                                  for dx, dy in dirs], dim=1))
    return torch.cat(S), torch.cat(J) if jac else None


def _gauss_newton64(meas, s, max_iter=20, tol=1e-6):
    B = meas.shape[0]
    lo, hi = (torch.from_numpy(v).to(DEV) for v in (s.lo, s.hi))
    th = torch.zeros((B, 4), dtype=torch.float64, device=DEV)
    th[:, 3] = 1.0
    live = torch.ones(B, dtype=torch.bool, device=DEV)
    for _ in range(max_iter):
        k = live.nonzero()[:, 0]
        if len(k) == 0:
            break
        S, J = _probe_slopes64(s, th[k], jac=True)
        r = meas[k].double() - S
        G = torch.stack([torch.stack([(J[:, a] * J[:, b]).sum(1) for b in range(4)], 1) for a in range(4)], 1)
        q = torch.stack([(J[:, a] * r).sum(1) for a in range(4)], 1)
        d = torch.linalg.solve(G.cpu(), q.cpu()).to(DEV)
        th[k] = torch.minimum(torch.maximum(th[k] + d, lo - (hi - lo) / 2), hi + (hi - lo) / 2)
        live[k] = (d / ((hi - lo) / 2)).square().sum(1).sqrt() >= tol
    return th


def _train64(case, seed):
    net, params, m, v, x, t = _train_state(case, seed)
    d = net.desc
    P = params.double()
    shapes = [(d.h1, d.n_in), (d.h1,), (d.h2, d.h1), (d.h2,), (d.n_out, d.h2), (d.n_out,)]
    W1, b1, W2, b2, W3, b3 = (q.reshape(sh) for q, sh in zip(P.split([math.prod(sh) for sh in shapes]), shapes))
    X = torch.zeros((x.shape[0], d.n_in), dtype=torch.float64, device=DEV)
    X[:, d.seg0:d.seg0 + d.len0] = x[:, :d.len0].double()
    X[:, d.seg1:d.seg1 + d.len1] = x[:, d.len0:].double()
    a1 = torch.relu(X @ W1.t() + b1)
    a2 = torch.relu(a1 @ W2.t() + b2)
    y = a2 @ W3.t() + b3
    dy = 2 * (y - t.double()) / y.numel()
    g2 = (dy @ W3) * (a2 > 0)
    g1 = (g2 @ W2) * (a1 > 0)
    grads = torch.cat([q.reshape(-1) for q in (g1.t() @ X, g1.sum(0), g2.t() @ a1, g2.sum(0), dy.t() @ a2, dy.sum(0))])
    b1_, b2_, eps, lr, step = 0.9, 0.999, 1e-8, 1e-4, 1001
    mm = b1_ * m.double() + (1 - b1_) * grads
    vv = b2_ * v.double() + (1 - b2_) * grads * grads
    new = P - lr * (mm / (1 - b1_ ** step)) / ((vv / (1 - b2_ ** step)).sqrt() + eps)
    return y, ((y - t.double()) ** 2).mean().reshape(1), grads, new, mm, vv


def _blocks(pupil, b):
    n = pupil.shape[0] // b
    return np.nonzero(pupil.reshape(n, b, n, b).any(axis=(1, 3)))


def _projection64(comps, dirs, pupil, pix, b):
    by, bx = _blocks(pupil, b)
    f = np.arange(b)
    yy = (by[:, None, None] * b + f[None, :, None]) + 0 * f[None, None, :]
    xx = (bx[:, None, None] * b + f[None, None, :]) + 0 * f[None, :, None]
    inside = torch.from_numpy(pupil[yy, xx].reshape(len(by), -1)).to(DEV).double()
    c = (pupil.shape[0] - 1) / 2.0
    ry = torch.from_numpy((yy.reshape(len(by), -1) - c) * pix).to(DEV)
    rx = torch.from_numpy((xx.reshape(len(by), -1) - c) * pix).to(DEV)
    w = inside / inside.sum(1, keepdim=True)
    out = []
    for F, h, s in comps:
        g = F.shape[1]
        P = torch.empty((F.shape[0], len(dirs), len(by)), dtype=torch.float64, device=DEV)
        for k, d in enumerate(dirs):
            taps = _taps((g - 1) / 2.0 + (rx + h * d[0]) / s, (g - 1) / 2.0 + (ry + h * d[1]) / s, g, g)
            for q in _chunks(F.shape[0], rx.numel() * 3):
                P[q, k] = (_gather(F[q], taps) * w).sum(-1)
        out.append(P.reshape(F.shape[0], -1))
    return torch.cat(out)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("im", "jacobian", "step", "warp"):
        F, theta, pupil, valid = _scao(case, seed)
        A, b, planes = _inverse(theta, case["grid"], pupil.shape[0])
        if kind == "im":
            mask = torch.from_numpy(_dm_mask(case)).to(DEV) if case["engine"] == "repaired" else None
            return _build64(F, A, b, pupil, case["p"], valid, engine=case["engine"], mask=mask)
        if kind == "warp":
            x, y = _window(pupil.shape[0])
            taps = _taps(*_points(A, b, x, y), case["grid"], case["grid"])
            phi = torch.cat([_gather(F[c], taps) for c in _chunks(F.shape[0], 4 * x.numel())])
            return phi, torch.cat([_differences(phi[c], pupil, case["p"], valid) for c in _chunks(F.shape[0], 4 * x.numel())])
        im, dim = _build64(F, A, b, pupil, case["p"], valid, planes=planes)
        if kind == "jacobian":
            return im, dim
        g = torch.randn(im.shape, generator=torch.Generator(device=DEV).manual_seed(int(seed)), device=DEV)
        return im, (dim * g.double()[None]).sum((1, 2)).cpu()
    if kind == "modal":
        F, g, pupil, valid = _modal(case, seed)
        return _build64(F, *_inverse_geometry(g, case["grid"], pupil.shape[0]), pupil, case["p"], valid)
    if kind == "mcao":
        stacks, wfs, geo = _mcao(case, seed)
        n_out = case["n_sub"] * case["p"]
        return [_build64(stacks[d], *_inverse_geometry(g, case["grid"], n_out), wfs[w][0], case["p"], wfs[w][1])
                for w, d, g in geo]
    if kind == "fit":
        meas, s = _probe_fit(case, seed)
        return _gauss_newton64(meas, s), None
    if kind == "train":
        return _train64(case, seed)
    dms, layers, dirs, pupil, pix, lam = _proj_inputs(case, seed)
    D = _projection64(dms, dirs, pupil, pix, case["bin"])
    L = _projection64(layers, dirs, pupil, pix, case["bin"])
    G = D @ D.t()
    G.diagonal().add_(lam)
    return torch.cholesky_solve(D @ L.t(), torch.linalg.cholesky(G))
