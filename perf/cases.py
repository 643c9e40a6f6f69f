"""Performance cases of the library: the work a program built on it has it do,
through the public entry points, from the smallest problem the library is used
on to the benchmark's 256^3 reconstruction.

A case is a dict of plain values.  `listed` gives the fixed cases, `draw` one
more of the same ranges, `prepare` what a program holds before the call
(inputs made from the seed alone, the built plan, buffers), `run` one pass,
`work` the bytes and operations a pass cannot do without, and `exact` what the
pass returns, computed in 64 bits by plain torch.

Inputs: a phantom of nested soft-edged ellipsoids; observed patches sampled
from it at the moved pixel positions (trilinear, averaged through the slice),
with 1 % noise and 10 % outlier patches; the current volume is a perturbed
phantom and the current motion the true one plus an error of up to 1 degree and
1 mm, the state between two cycles of a reconstruction.
"""
import math

import numpy as np
import torch

from paper_1611_07289_amd import autograd, batch, driver, learned, pvr, superpixel, synth

K = 3.0  # PSF support radius (standard deviations)
FWHM = (1.0, 1.0, 4.0)

# The convolutions of the learned initialiser: (cin, cout, stride, input side)
LAYERS = ((2, 32, 1, 64), (32, 32, 2, 64), (32, 64, 1, 32), (64, 64, 2, 32), (64, 64, 1, 16),
          (64, 64, 2, 16), (64, 64, 1, 8), (64, 64, 1, 8))


def listed():
    return [
        # the smallest reconstruction (32^3, 16-pixel patches): launches and latency
        {"name": "sr_tiny32", "kind": "sr", "nx": 32, "ny": 32, "nz": 32, "slices": 8, "a": 16,
         "stacks": 3, "psf": "gauss"},
        # the benchmark's SR iteration: 256^3, 4 stacks, 11 760 patches, 48 M samples
        {"name": "sr_256", "kind": "sr", "nx": 256, "ny": 256, "nz": 256, "slices": 60, "a": 64,
         "stacks": 4, "psf": "gauss"},
        # the forward pass alone at ragged sizes: odd grid, odd patches cut from odd slices
        {"name": "forward_ragged", "kind": "forward", "nx": 149, "ny": 131, "nz": 117,
         "slices": 31, "a": 37, "stacks": 4, "psf": "gauss"},
        # what follows every registration pass: the build at the new motion, the adjoint's
        # index, and the first volume A^T y / A^T 1
        {"name": "rebuild_160", "kind": "rebuild", "nx": 160, "ny": 160, "nz": 160, "slices": 40,
         "a": 64, "stacks": 4, "psf": "gauss"},
        # several independent reconstructions in one plan, SR iterations replayed as a graph
        {"name": "batch_graph", "kind": "batch", "n0": 96, "n1": 126, "n2": 150, "a0": 32,
         "a1": 64, "a2": 128},
        # an SR iteration with the paper's sinc PSF
        {"name": "sr_sinc_128", "kind": "sr", "nx": 128, "ny": 128, "nz": 128, "slices": 32,
         "a": 64, "stacks": 4, "psf": "sinc"},
        # differentiable simulation, forward and backward, in FP32 and FP64
        {"name": "grad_f32_96", "kind": "grad", "nx": 96, "ny": 96, "nz": 96, "slices": 24,
         "a": 32, "stacks": 3, "f64": False},
        {"name": "grad_f64_48", "kind": "grad", "nx": 48, "ny": 48, "nz": 48, "slices": 12,
         "a": 24, "stacks": 3, "f64": True},
        # refinement of every patch's motion (the budget used after the learned initialiser)
        {"name": "register_128", "kind": "register", "nx": 128, "ny": 128, "nz": 128,
         "slices": 32, "a": 64, "stacks": 4, "exact_gradient": True, "steps": 5, "psf": "gauss"},
        # superpixel patches of a whole acquisition: clustering, dilation, packing
        {"name": "superpixel_256", "kind": "superpixel", "images": 240, "h": 256, "w": 256,
         "a": 32, "gamma": 19, "iters": 10},
        # the learned initialiser: one batch of predictions, and one layer in training
        {"name": "cnn_predict_1024", "kind": "predict", "batch": 1024},
        {"name": "cnn_layer_256", "kind": "layer", "layer": 2, "batch": 256},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sr", "sr", "forward", "rebuild", "batch", "grad", "register",
                       "superpixel", "predict", "layer"])
    if kind == "batch":
        c = {"kind": kind}
        for i in range(3):
            c["n%d" % i] = rng.randint(64, 160)
            c["a%d" % i] = rng.choice([32, 48, 64, 128])
        return c
    if kind == "superpixel":
        a = rng.choice([16, 24, 32, 64])
        return {"kind": kind, "images": _log(rng, 8, 240), "h": rng.randint(96, 256),
                "w": rng.randint(96, 256), "a": a, "gamma": int(0.6 * a),
                "iters": rng.choice([5, 10])}
    if kind == "predict":
        return {"kind": kind, "batch": _log(rng, 16, 1024)}
    if kind == "layer":
        return {"kind": kind, "layer": rng.randint(1, len(LAYERS) - 1),
                "batch": _log(rng, 16, 512)}
    hi = {"sr": 224, "forward": 224, "rebuild": 208, "grad": 128, "register": 160}[kind]
    n = _log(rng, 32, hi)
    c = {"kind": kind}
    for ax in ("nx", "ny", "nz"):
        c[ax] = min(hi, max(24, int(n * rng.uniform(0.85, 1.15))))
    c["slices"] = max(4, n // 4)
    c["a"] = min(rng.choice([16, 32, 64, rng.randint(17, 64)]), n // 2)
    c["stacks"] = rng.randint(3, 5)
    if kind in ("sr", "forward", "rebuild"):
        c["psf"] = rng.choice(["gauss", "gauss", "sinc"])
    if kind == "grad":
        c["f64"] = rng.random() < 0.4
        if c["f64"]:
            c.update(nx=min(c["nx"], 64), ny=min(c["ny"], 64), nz=min(c["nz"], 64),
                     slices=min(c["slices"], 16), a=min(c["a"], 24))
    if kind == "register":
        c["exact_gradient"] = rng.random() < 0.6
        c["steps"] = rng.choice([1, 3, 5])
        c["psf"] = "gauss" if c["exact_gradient"] or rng.random() < 0.6 else "sinc"
    return c


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------
def _gpu():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gen(seed):
    return torch.Generator(device=_gpu()).manual_seed(int(seed) % (1 << 62))


class _Problem:
    """One reconstruction's geometry, motion, phantom and observations."""

    def __init__(self, nx, ny, nz, slices, a, stacks, seed):
        rng = np.random.default_rng([int(seed), 1])
        v2w = np.zeros((3, 4))
        v2w[0, 0] = v2w[1, 1] = v2w[2, 2] = 1.0
        self.grid = synth.Grid(nx, ny, nz, v2w)
        c = synth.grid_center(self.grid)
        self.stacks, parts = [], []
        frames = synth.orthogonal_frames([30.0, 50.0, 20.0][:max(0, stacks - 3)])
        for i, fr in enumerate(frames[:stacks]):
            # in-plane extents follow the grid axes the stack's axes run along
            n1 = (nx, nx, ny)[i] if i < 3 else nx
            n2 = (ny, nz, nz)[i] if i < 3 else ny
            st = synth.make_stack(c, *fr, n1, n2, slices, (1, 1), 4.0, FWHM)
            self.stacks.append(st)
            parts.append(synth.square_patches([st], a, max(1, a // 2), stack_base=i))
        self.parts = parts
        self.patches = synth.concat_patches(parts)
        M = self.patches.M
        self.theta_true = synth.random_motion_batch(M, 10.0, 5.0, int(rng.integers(1 << 30)))
        err = synth.random_motion_batch(M, 1.0, 1.0, int(rng.integers(1 << 30)))
        self.theta = (self.theta_true + err).astype(np.float32)
        self.outlier = rng.random(M) < 0.10
        self.seed = int(seed)
        self.X_true = _phantom(nx, ny, nz, rng)

    def observe(self):
        """y [N] float32: the phantom at the moved pixels, noise, outliers."""
        g = _gen(self.seed * 7 + 3)
        out, top, s0 = [], float(self.X_true.max()), 0
        X5 = self.X_true[None, None]
        size = torch.tensor([X5.shape[4], X5.shape[3], X5.shape[2]], device=_gpu())
        for st, part in zip(self.stacks, self.parts):
            M = part.M
            A = torch.from_numpy(_moved(st, part, self.theta_true[s0:s0 + M])).to(_gpu())
            pix = _pixels(part)
            y = torch.zeros(M, pix.shape[1], device=_gpu())
            for dn, wt in ((-0.3, 0.25), (0.0, 0.5), (0.3, 0.25)):
                q = pix.clone()
                q[..., 2] += dn
                x = torch.einsum("mrc,mpc->mpr", A[:, :, :3], q) + A[:, None, :, 3]
                x = (2.0 * x / (size - 1) - 1.0).float()
                y += wt * torch.nn.functional.grid_sample(
                    X5, x[None, :, :, None], mode="bilinear", padding_mode="zeros",
                    align_corners=True)[0, 0, :, :, 0]
            y += 0.01 * top * torch.randn(y.shape, generator=g, device=_gpu())
            bad = torch.from_numpy(self.outlier[s0:s0 + M]).to(_gpu())
            noise = top * torch.rand(y.shape, generator=g, device=_gpu())
            out.append(torch.where(bad[:, None], noise, y).reshape(-1))
            s0 += M
        return torch.cat(out)

    def volume(self):
        """The current volume [V] float32: the phantom, perturbed."""
        g = _gen(self.seed * 7 + 4)
        X = self.X_true * (1 + 0.05 * torch.randn(self.X_true.shape, generator=g, device=_gpu()))
        return X.clamp_(min=0).reshape(-1).contiguous()


def _phantom(nx, ny, nz, rng):
    dev = _gpu()
    z, y, x = torch.meshgrid(*(torch.arange(n, device=dev, dtype=torch.float32)
                               for n in (nz, ny, nx)), indexing="ij")
    n = np.array([nx, ny, nz], float)
    vol = torch.zeros(nz, ny, nx, device=dev)

    def paint(c, semi, R, value):
        d = [x - float(c[0]), y - float(c[1]), z - float(c[2])]
        q = sum((sum(float(R[r, k]) * d[r] for r in range(3)) / float(semi[k])) ** 2
                for k in range(3))
        soft = torch.sigmoid((1 - q.sqrt()) * float(np.mean(semi)))
        vol.lerp_(torch.full_like(vol, value), soft)

    c0 = (n - 1) / 2
    semi0 = np.array([0.43, 0.35, 0.31]) * n
    paint(c0, semi0, np.eye(3), 400.0)
    for e in range(5):
        semi = rng.uniform(0.05, 0.16, size=3) * n
        c = c0 + rng.uniform(-0.5, 0.5, size=3) * (semi0 - semi.max())
        paint(c, semi, synth.random_rotation(rng), (200.0, 600.0, 1000.0)[e % 3])
    return vol


def _rotations(th):
    cx, sx = np.cos(th[:, 0]), np.sin(th[:, 0])
    cy, sy = np.cos(th[:, 1]), np.sin(th[:, 1])
    cz, sz = np.cos(th[:, 2]), np.sin(th[:, 2])
    R = np.empty((th.shape[0], 3, 3))
    R[:, 0] = np.stack([cz * cy, cz * sy * sx - sz * cx, cz * sy * cx + sz * sx], 1)
    R[:, 1] = np.stack([sz * cy, sz * sy * sx + cz * cx, sz * sy * cx - cz * sx], 1)
    R[:, 2] = np.stack([-sy, cy * sx, cy * cx], 1)
    return R


def _centres(st, part):
    pc = np.stack([part.x0 + 0.5 * (part.w - 1), part.y0 + 0.5 * (part.h - 1),
                   part.slice], 1).astype(float)
    P = np.asarray(st.pix2world, float)
    return pc @ P[:, :3].T + P[:, 3]


def _moved(st, part, theta):
    """[M][3][4]: pixel (u, v, slice) -> voxel of the moved sample centre
    (the grid's voxels are 1 mm and start at the world's origin)."""
    th = np.asarray(theta, float)
    R, c = _rotations(th), _centres(st, part)
    P = np.asarray(st.pix2world, float)
    A = np.empty((th.shape[0], 3, 4))
    A[:, :, :3] = R @ P[:, :3]
    A[:, :, 3] = np.einsum("mrc,mc->mr", R, P[:, 3] - c) + c + th[:, 3:]
    return A


def _pixels(part):
    """[M][w h][3] float64 pixel coordinates of a part's samples (one size)."""
    w, h = int(part.w[0]), int(part.h[0])
    u, v = np.meshgrid(np.arange(w), np.arange(h), indexing="xy")
    uv = torch.from_numpy(np.stack([u.ravel(), v.ravel()], 1).astype(float)).to(_gpu())
    o = torch.from_numpy(np.stack([part.x0, part.y0], 1).astype(float)).to(_gpu())
    p = torch.empty(part.M, w * h, 3, dtype=torch.float64, device=_gpu())
    p[..., :2] = uv[None] + o[:, None]
    p[..., 2] = torch.from_numpy(part.slice.astype(float)).to(_gpu())[:, None]
    return p


def _problem(case, seed):
    return _Problem(case["nx"], case["ny"], case["nz"], case["slices"], case["a"],
                    case["stacks"], seed)


def _batch_problems(case, seed):
    return [_Problem(n, n, n, -(-n // 4), min(a, n), 3 + i, 31 * seed + i)
            for i, (n, a) in enumerate((case["n%d" % i], case["a%d" % i]) for i in range(3))]


def _images(case, seed):
    """[n][h][w]: slices through the middle of a phantom, with noise."""
    n, h, w = case["images"], case["h"], case["w"]
    V = _phantom(w, h, n, np.random.default_rng([int(seed), 2]))
    return (V + 10.0 * torch.randn(V.shape, generator=_gen(seed * 7 + 5), device=_gpu())).contiguous()


def _layer_inputs(case, seed):
    cin, cout, s, side = LAYERS[case["layer"]]
    B, so = case["batch"], (side - 1) // s + 1
    g = _gen(seed * 7 + 6)

    def rnd(*shape):
        return torch.randn(*shape, generator=g, device=_gpu())
    w = rnd(cout, 3, 3, cin) * math.sqrt(2.0 / (9 * cin))
    return {"x": rnd(B, side, side, cin).clamp_(min=0).bfloat16(), "w": w.bfloat16(),
            "bias": 0.1 * rnd(cout), "gout": (0.01 * rnd(B, so, so, cout)).bfloat16()}


def _pairs(case, seed):
    """Observed and simulated 64 x 64 patches [B][64][64] (float32)."""
    B = case["batch"]
    g = _gen(seed * 7 + 8)
    V = _phantom(96, 96, 64, np.random.default_rng([int(seed), 3]))
    ox, oy = (torch.randint(0, 33, (B,), generator=g, device=_gpu()) for _ in range(2))
    oz = torch.randint(8, 56, (B,), generator=g, device=_gpu())
    i = torch.arange(64, device=_gpu())
    y = V[oz[:, None, None], (oy[:, None] + i)[:, :, None], (ox[:, None] + i)[:, None, :]]
    ys = torch.roll(y, (1, 2), (1, 2))
    return (y + 10.0 * torch.randn(y.shape, generator=g, device=_gpu())).contiguous(), \
        (ys + 1e-2 * torch.randn(y.shape, generator=g, device=_gpu())).contiguous()


def _built(probs, psf="gauss", f64=False):
    plan = pvr.Plan.from_problems(probs, K, f64=f64)
    if psf == "sinc":
        plan.set_psf(pvr.PVR_PSF_SINC)
    theta = torch.from_numpy(np.concatenate([p.theta for p in probs])).to(_gpu())
    plan.build(theta.double() if f64 else theta)
    return plan, theta


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "superpixel":
        s["img"] = _images(case, seed)
        # buffers for the packed patches, with room for the dilated boxes
        n = int(2.5 * s["img"].numel() * (1 + 2 * case["gamma"] / case["a"]) ** 2)
        s["y"] = torch.zeros(n, device=_gpu())
        s["mask"] = torch.zeros(n, dtype=torch.uint8, device=_gpu())
        k = case["images"] * superpixel.n_centres(case["h"], case["w"], case["a"])
        s["ws"] = torch.empty(pvr.load().pvr_slic_pack_workspace(k), dtype=torch.uint8,
                              device=_gpu())
        return s
    if kind == "layer":
        s.update(_layer_inputs(case, seed))
        cin, cout, st, side = LAYERS[case["layer"]]
        B = case["batch"]
        s["wt"] = s["w"].permute(1, 2, 3, 0).contiguous()
        s["out"] = torch.empty_like(s["gout"])
        s["gin"] = torch.empty_like(s["x"])
        s["dw"] = torch.empty(cout, 3, 3, cin, device=_gpu())
        s["db"] = torch.empty(cout, device=_gpu())
        n = pvr.load().pvr_cnn_wgrad_scratch(B, side, side, cin, cout, st)
        s["scratch"] = torch.empty(n // 4 + 16, device=_gpu())
        return s
    if kind == "predict":
        B = case["batch"]
        # one patch per slice, at rest in the middle of the grid: every sample valid
        g = synth.iso_grid(96)
        st = synth.make_stack(synth.grid_center(g), *np.eye(3), 64, 64, B, (1, 1), 60.0 / B, FWHM)
        s["plan"] = pvr.Plan([g], [[st]], [synth.square_patches([st], 64, 64)], K)
        s["plan"].build(torch.zeros(B, 6, device=_gpu()))
        y, ys = _pairs(case, seed)
        s["y"], s["ysim"] = y.reshape(-1), ys.reshape(-1)
        s["ids"] = torch.arange(B, dtype=torch.int32, device=_gpu())
        s["net"] = learned.Net(seed=int(seed) % (1 << 31))
        s["net"].buffers(B)
        return s
    if kind == "batch":
        probs = _batch_problems(case, seed)
        s["plan"], s["theta"] = _built(probs)
        y = torch.cat([p.observe() for p in probs])
        s["X"] = torch.cat([p.volume() for p in probs])
        s["sr"] = batch.GraphedSR(s["plan"], y, s["X"])
        s["sr"].start()
        s["sr"].capture()
        return s
    f64 = bool(case.get("f64"))
    prob = _problem(case, seed)
    s["plan"], s["theta"] = _built([prob], case.get("psf", "gauss"), f64)
    s["X"] = prob.volume()
    if kind == "grad":
        dt = torch.float64 if f64 else torch.float32
        s["X"] = s["X"].to(dt).requires_grad_()
        s["theta"] = s["theta"].to(dt).requires_grad_()
        s["gy"] = torch.randn(s["plan"].N, generator=_gen(seed * 7 + 9), device=_gpu()).to(dt)
        return s
    s["y"] = prob.observe()
    if kind == "register":
        s["ncc"] = torch.empty(s["plan"].M, device=_gpu())
        s["params"] = pvr.RegParams.make(step0=0.25, max_iter=case["steps"],
                                         min_std=0.01 * float(s["y"].abs().max()),
                                         exact=case["exact_gradient"])
    else:
        s["buf"] = driver.Buffers(s["plan"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "superpixel":
        img, a, gamma = s["img"], case["a"], case["gamma"]
        lab, C = superpixel.slic(img, a, 40.0, 5.0, case["iters"])
        B = superpixel.boxes(lab, C, a, gamma).cpu().numpy()
        tab = np.ascontiguousarray(superpixel.patch_table(B))
        assert int((tab[:, 4].astype(np.int64) * tab[:, 5]).sum()) <= s["y"].numel()
        pvr._check(pvr.load().pvr_slic_pack(
            img.data_ptr(), lab.data_ptr(), *img.shape, gamma, tab.shape[0], tab.ctypes.data,
            s["ws"].data_ptr(), s["ws"].numel(), s["y"].data_ptr(), s["mask"].data_ptr(),
            torch.cuda.current_stream().cuda_stream))
        return {"labels": lab, "centres": C, "boxes": B, "y": s["y"], "mask": s["mask"]}
    if kind == "layer":
        cin, cout, st, side = LAYERS[case["layer"]]
        B, L, q = case["batch"], pvr.load(), torch.cuda.current_stream().cuda_stream
        p = {k: s[k].data_ptr() for k in ("x", "w", "wt", "bias", "gout", "out", "gin", "dw",
                                          "db", "scratch")}
        pvr._check(L.pvr_cnn_conv_fwd(p["x"], p["w"], p["bias"], p["out"], B, side, side, cin,
                                      cout, st, 1, q))
        pvr._check(L.pvr_cnn_conv_wgrad(p["gout"], p["out"], p["x"], p["scratch"], p["dw"],
                                        p["db"], B, side, side, cin, cout, st, q))
        pvr._check(L.pvr_cnn_conv_dgrad(p["gout"], p["out"], p["wt"], p["gin"], B, side, side,
                                        cin, cout, st, q))
        return {k: s[k] for k in ("out", "gin", "dw", "db")}
    if kind == "predict":
        return s["net"].predict(s["plan"], s["y"], s["ysim"], s["ids"], case["batch"])
    plan, X = s["plan"], s["X"]
    if kind == "batch":
        sr = s["sr"]
        sr.replay_pairs(1)
        return {"X": sr.X, "e": sr.e, "p": sr.p, "W": sr.W, "num": sr.num, "den": sr.den}
    if kind == "grad":
        y = autograd.simulate(X, s["theta"], plan)
        gX, gth = torch.autograd.grad(y, (X, s["theta"]), s["gy"])
        return {"y": y.detach(), "gX": gX, "gtheta": gth}
    if kind == "register":
        theta = s["theta"].clone()
        plan.register(X, s["y"], theta, s["ncc"], params=s["params"])
        return {"theta": theta, "ncc": s["ncc"]}
    y, b = s["y"], s["buf"]
    if kind == "rebuild":
        plan.build(s["theta"])
        X0 = driver.initial_volume(plan, y, b)
        return {"X0": X0, "num": b.num, "den": b.den}
    if kind == "forward":
        plan.simulate(X, y_obs=y, resid=b.e)
        return b.e
    plan.simulate(X, y_obs=y, resid=b.e)
    plan.robust_weights(b.e, y, b.em, b.p, b.pbar, b.W, pvr.PVR_EM_INIT
                        | pvr.PVR_EM_RESID_FRESH | pvr.PVR_EM_PREP_ADJOINT)
    plan.backproject(b.e, b.p, b.W, b.num, b.den)
    plan.sr_update(X, b.num, b.den, b.Xn)
    return {"X": b.Xn, "e": b.e, "p": b.p, "pbar": b.pbar, "W": b.W, "num": b.num, "den": b.den}


# ----------------------------------------------------------------------------
# work: inputs read once, outputs written once, and the PSF's nonzeros
# ----------------------------------------------------------------------------
def _sizes(nx, ny, nz, slices, a, stacks):
    """(samples, patches, voxels) of a problem."""
    N = M = 0
    for i in range(stacks):
        n1 = (nx, nx, ny)[i] if i < 3 else nx
        n2 = (ny, nz, nz)[i] if i < 3 else ny
        w, h = min(a, n1), min(a, n2)
        m = slices * len(range(0, n1 - w + 1, max(1, min(a // 2, w)))) \
            * len(range(0, n2 - h + 1, max(1, min(a // 2, h))))
        M += m
        N += m * w * h
    return N, M, nx * ny * nz


def work(case):
    kind = case["kind"]
    if kind == "superpixel":
        n = case["images"] * case["h"] * case["w"]
        packed = n * (1 + 2 * case["gamma"] / case["a"]) ** 2
        # a pixel is compared with the 4 centres whose window covers it, every round
        return {"bytes": 8.0 * n + 5.0 * packed, "flops": 4.0 * 8 * n * (case["iters"] + 1)}
    if kind == "layer":
        cin, cout, st, side = LAYERS[case["layer"]]
        B, so = case["batch"], (side - 1) // st + 1
        act = 2.0 * B * (side * side * cin * 2 + so * so * cout * 2)
        return {"bytes": act + 8.0 * 9 * cin * cout, "flops": 3 * 2.0 * B * so * so * cout * 9 * cin}
    if kind == "predict":
        return {"bytes": case["batch"] * (64 * 64 * 8.0 + 24) + 4e5,
                "flops": 2.0 * case["batch"] * learned.macs_per_pair()}
    if kind == "batch":
        N = M = V = 0
        for i in range(3):
            n = case["n%d" % i]
            x = _sizes(n, n, n, -(-n // 4), min(case["a%d" % i], n), 3 + i)
            N, M, V = N + x[0], M + x[1], V + x[2]
    else:
        N, M, V = _sizes(case["nx"], case["ny"], case["nz"], case["slices"], case["a"],
                         case["stacks"])
    s = [f / 2.3548 for f in FWHM]
    nnz = N * (4.0 / 3.0 * math.pi * K ** 3 * s[0] * s[1] * s[2])
    if case.get("psf") == "sinc":
        nnz = N * 2.0 * 2.0 * 2 * K * s[2]
        fwd, adj = 51.0 * nnz, 52.0 * nnz
    else:
        fwd, adj = 16.0 * nnz, 17.0 * nnz
    if kind == "forward":
        return {"bytes": 4.0 * V + 8.0 * N, "flops": fwd}
    if kind == "rebuild":
        return {"bytes": 12.0 * V + 4.0 * N, "flops": fwd + adj}
    if kind == "grad":
        b = 8.0 if case["f64"] else 4.0
        return {"bytes": b * (2 * V + 2 * N), "flops": 2 * fwd + 2 * adj}
    if kind == "register":
        g = 2.3 if case["exact_gradient"] else 12.0
        return {"bytes": 4.0 * (V + N) + 52.0 * M, "flops": fwd * (1 + case["steps"] * (1 + 0.5 * g))}
    iters = 2 if kind == "batch" else 1  # the reads and writes of a patch's samples and the volume
    return {"bytes": iters * (16.0 * V + 12.0 * N), "flops": iters * (fwd + adj)}


# ----------------------------------------------------------------------------
# exact: the same in 64 bits, by plain torch
# ----------------------------------------------------------------------------
CHUNK = 1 << 25  # sample-voxel pairs at a time


def _supports(prob, psf):
    """For a few patches at a time: (first sample, number, voxel index [n][B],
    weight g [n][B], normaliser Z [n] (0: invalid), in-support voxel offsets
    D [n][B][3], per-sample patch, patch geometry)."""
    dev = _gpu()
    nx, ny, nz = prob.grid.nx, prob.grid.ny, prob.grid.nz
    size = torch.tensor([nx, ny, nz], device=dev, dtype=torch.float64)
    s0 = j0 = 0
    cut = math.exp(-0.5 * K * K)
    sig = np.array(FWHM) / (2.0 * math.sqrt(2.0 * math.log(2.0)))
    for st, part in zip(prob.stacks, prob.parts):
        M = part.M
        th = np.asarray(prob.theta[s0:s0 + M], float)
        A = torch.from_numpy(_moved(st, part, th)).to(dev)
        P = np.asarray(st.pix2world, float)[:, :3]
        F = _rotations(th) @ (P / np.linalg.norm(P, axis=0))
        if psf == "sinc":
            ext = np.abs(F) @ np.array([FWHM[0], FWHM[1], K * sig[2]])
        else:
            ext = K * np.sqrt((F ** 2) @ (sig ** 2))
        hw = np.floor(ext.max(axis=0) + 0.5).astype(int)
        o = torch.stack(torch.meshgrid(*(torch.arange(-h, h + 1, device=dev, dtype=torch.float64)
                                         for h in hw), indexing="ij"), -1).reshape(-1, 3)
        Ft = torch.from_numpy(F).to(dev)
        pix = _pixels(part)
        n1 = pix.shape[1]
        step = max(1, CHUNK // (n1 * o.shape[0]))
        sg = torch.from_numpy(sig).to(dev)
        for a in range(0, M, step):
            m = min(step, M - a)
            x = torch.einsum("mrc,mpc->mpr", A[a:a + m, :, :3], pix[a:a + m]) + A[a:a + m, None, :, 3]
            b = torch.round(x)
            D = (b - x)[:, :, None, :] + o                      # [m][p][B][3]
            v = b[:, :, None, :] + o
            ok = ((v >= 0) & (v <= size - 1)).all(-1)
            t = torch.einsum("mpbr,mra->mpba", D, Ft[a:a + m])  # along the stack axes (mm)
            if psf == "sinc":
                tu, tv = t[..., 0] / FWHM[0], t[..., 1] / FWHM[1]
                gz = (torch.exp(-0.5 * (t[..., 2] / sg[2]) ** 2) - cut).clamp_(min=0)
                g = torch.sinc(tu) * torch.sinc(tv) * gz
                g = torch.where(ok & (tu.abs() < 1) & (tv.abs() < 1), g, 0.0)
                e2 = None
            else:
                Q = ((t / sg) ** 2).sum(-1)
                e2 = torch.where(ok & (Q <= K * K), torch.exp(-0.5 * Q), 0.0)
                g = torch.where(e2 > 0, e2 - cut, 0.0).clamp_(min=0)
            Z = g.sum(-1)
            inside = ((x >= -0.5) & (x < size - 0.5)).all(-1)
            Z = torch.where(inside, Z, 0.0)
            vi = torch.where(ok[..., None], v, 0.0).long()
            idx = (vi[..., 2] * ny + vi[..., 1]) * nx + vi[..., 0]
            yield (j0 + a * n1, s0 + a, m, n1, idx, g, Z, e2, D, x, Ft[a:a + m], part, a, st, th)
        s0 += M
        j0 += M * n1


def _forward64(prob, X, psf="gauss"):
    """(A X [N], valid [N])"""
    ys, va = [], []
    for _, _, m, n1, idx, g, Z, *_ in _supports(prob, psf):
        y = (g * X[idx]).sum(-1)
        ys.append(torch.where(Z > 0, y / Z.clamp(min=1e-300), 0.0).reshape(-1))
        va.append((Z > 0).reshape(-1))
    return torch.cat(ys), torch.cat(va)


def _adjoint64(prob, r, q, psf="gauss"):
    """sum_j psi_ji r_j and sum_j psi_ji q_j over the voxels [V]."""
    V = prob.grid.n_voxels
    num = torch.zeros(V, dtype=torch.float64, device=_gpu())
    den = torch.zeros_like(num)
    for j, _, m, n1, idx, g, Z, *_ in _supports(prob, psf):
        iz = torch.where(Z > 0, 1.0 / Z.clamp(min=1e-300), 0.0)
        psi = g * iz[..., None]
        on = psi > 0
        at = idx[on]
        for out, val in ((num, r), (den, q)):
            if val is not None:
                out.index_add_(0, at, (psi * val[j:j + m * n1].reshape(m, n1, 1))[on])
    return num, den


def _em64(prob, e, y, valid, state):
    """One robust-weights call (state None starts EM): p, pbar, W, state."""
    M = prob.patches.M
    n = torch.from_numpy((prob.patches.w * prob.patches.h).astype(np.int64)).to(_gpu())
    pid = torch.repeat_interleave(torch.arange(M, device=_gpu()), n)
    v = valid.double()

    def per_patch(a):
        return torch.zeros(M, dtype=torch.float64, device=_gpu()).index_add_(0, pid, a * v)
    ev, yv = e[valid], y[valid].double()
    ymax = float(yv.abs().max())
    m = 1.0 / max(float(ev.max() - ev.min()), 1e-6 * ymax)
    floor2 = (1e-4 * ymax) ** 2
    s2, c = state or (max(float((ev * ev).mean()), floor2), 0.9)
    G = c / math.sqrt(2 * math.pi * s2) * torch.exp(-e * e / (2 * s2))
    p = G / (G + m * (1 - c)) * v
    ns, sp, sp2, spe2 = per_patch(torch.ones_like(p)), per_patch(p), per_patch(p * p), \
        per_patch(p * e * e)
    pbar = torch.where(ns > 0, (sp2 / ns.clamp(min=1)).sqrt(), 0.0)
    used = ns > 0
    x = torch.sort(pbar[used])[0]
    k = x.numel() // 2
    mu0, mu1 = x[:k].mean(), x[k:].mean()
    sd0, sd1 = x[:k].std(correction=0).clamp(min=1e-3), x[k:].std(correction=0).clamp(min=1e-3)
    w1 = torch.tensor(0.9, dtype=torch.float64, device=_gpu())

    def resp(t):
        l1 = torch.log(w1) - torch.log(sd1) - (t - mu1) ** 2 / (2 * sd1 ** 2)
        l0 = torch.log(1 - w1) - torch.log(sd0) - (t - mu0) ** 2 / (2 * sd0 ** 2)
        return torch.sigmoid(l1 - l0)
    for _ in range(20):
        r = resp(x)
        r1, r0 = r.sum(), (1 - r).sum()
        if not (float(r1) > 0 and float(r0) > 0):
            break
        mu1, mu0 = (r * x).sum() / r1, ((1 - r) * x).sum() / r0
        sd1 = ((r * (x - mu1) ** 2).sum() / r1).sqrt().clamp(min=1e-3)
        sd0 = (((1 - r) * (x - mu0) ** 2).sum() / r0).sqrt().clamp(min=1e-3)
        w1 = r1 / x.numel()
    pi = resp(pbar)
    pi = 1 - pi if float(mu0) > float(mu1) else pi
    W = torch.where(used & (pi >= 0.5), pi, 0.0)
    swp = float((W * sp).sum())
    return p, pbar, W, pid, (max(float((W * spe2).sum()) / swp, floor2), swp / float((W * ns).sum()))


def _update64(prob, X, num, den, lam=0.02, delta=150.0, clamp=True):
    nz, ny, nx = prob.grid.nz, prob.grid.ny, prob.grid.nx
    x = X.reshape(nz, ny, nx)
    step = torch.where(den > 1e-6, num / den.clamp(min=1e-300), 0.0).reshape(nz, ny, nx)
    R = torch.zeros_like(x)
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                if not (dx or dy or dz) or lam == 0.0:
                    continue
                src = tuple(slice(max(0, d), n + min(0, d)) for d, n in zip((dz, dy, dx), x.shape))
                dst = tuple(slice(max(0, -d), n + min(0, -d)) for d, n in zip((dz, dy, dx), x.shape))
                D = x[src] - x[dst]
                R[dst] += D / torch.sqrt(1 + (D / delta) ** 2) / math.sqrt(dx * dx + dy * dy + dz * dz)
    out = x + step + lam * R
    return (out.clamp(min=0) if clamp else out).reshape(-1)


def _sr64(prob, X, y, psf, state=None):
    ys, valid = _forward64(prob, X, psf)
    e = torch.where(valid, y.double() - ys, 0.0)
    p, pbar, W, pid, state = _em64(prob, e, y, valid, state)
    wp = p * W[pid]
    num, den = _adjoint64(prob, wp * e, wp, psf)
    return {"X": _update64(prob, X, num, den), "e": e, "p": p, "pbar": pbar, "W": W, "num": num,
            "den": den}, state


def _grad64(prob, X, gy):
    """y, d/dX and d/dtheta of sum gy y."""
    dev = _gpu()
    ys, _ = _forward64(prob, X)
    gX, _ = _adjoint64(prob, gy, None)
    gth = torch.zeros(prob.patches.M, 6, dtype=torch.float64, device=dev)
    sig = torch.tensor(FWHM, dtype=torch.float64, device=dev) / (2 * math.sqrt(2 * math.log(2.0)))
    for j, s, m, n1, idx, g, Z, e2, D, x, F, part, a, st, th in _supports(prob, "gauss"):
        iz = torch.where(Z > 0, 1.0 / Z.clamp(min=1e-300), 0.0)
        yh = ys[j:j + m * n1].reshape(m, n1, 1)
        wt = e2 * (X[idx] - yh) * (iz * gy[j:j + m * n1].reshape(m, n1))[..., None]
        Mq = (F / sig ** 2) @ F.transpose(1, 2)
        z = torch.einsum("mrc,mpbc->mpbr", Mq, D)
        t = torch.from_numpy(th[a:a + m]).to(dev)
        c = torch.from_numpy(_centres(st, part)[a:a + m]).to(dev)
        Y = D + (x - (c + t[:, 3:])[:, None])[:, :, None]
        cr = torch.einsum("mpb,mpbr->mr", wt, torch.linalg.cross(z, Y))
        cz, sz, cy, sy = torch.cos(t[:, 2]), torch.sin(t[:, 2]), torch.cos(t[:, 1]), torch.sin(t[:, 1])
        om = torch.zeros(m, 3, 3, dtype=torch.float64, device=dev)
        om[:, 0] = torch.stack([cz * cy, sz * cy, -sy], 1)
        om[:, 1] = torch.stack([-sz, cz, torch.zeros_like(cz)], 1)
        om[:, 2, 2] = 1.0
        gth[s:s + m, :3] = -torch.einsum("mkr,mr->mk", om, cr)
        gth[s:s + m, 3:] = torch.einsum("mpb,mpbr->mr", wt, z)
    return {"y": ys, "gX": gX, "gtheta": gth}


def _taps(x, st):
    """[B][H][W][C] -> [B][Ho][Wo][9][C] of the 3 x 3 windows (zero padded)."""
    B, H, W, C = x.shape
    xp = torch.zeros(B, H + 2, W + 2, C, dtype=x.dtype, device=x.device)
    xp[:, 1:-1, 1:-1] = x
    return torch.stack([xp[:, i:i + H:st, j:j + W:st] for i in range(3) for j in range(3)], 3)


def _conv64(x, w, b, st):
    """relu(conv3x3(x) + b), w [cout][9 cin], a few images at a time."""
    out = []
    for i in range(0, x.shape[0], 64):
        t = _taps(x[i:i + 64].double(), st)
        out.append((t.flatten(3) @ w.double().T + b.double()).clamp(min=0))
    return torch.cat(out)


def _layer64(case, seed):
    cin, cout, st, side = LAYERS[case["layer"]]
    d = _layer_inputs(case, seed)
    w = d["w"].double()
    out = _conv64(d["x"], w.reshape(cout, -1), d["bias"], st)
    g = torch.where(out > 0, d["gout"].double(), 0.0)
    dw = torch.zeros(cout, 9 * cin, dtype=torch.float64, device=_gpu())
    gin = torch.zeros(case["batch"], side + 2, side + 2, cin, dtype=torch.float64, device=_gpu())
    for i in range(0, case["batch"], 64):
        gi = g[i:i + 64].reshape(-1, cout)
        dw += gi.T @ _taps(d["x"][i:i + 64].double(), st).flatten(3).reshape(-1, 9 * cin)
        gt = (g[i:i + 64] @ w.reshape(cout, -1)).unflatten(-1, (9, cin))
        for k in range(9):
            gin[i:i + 64, k // 3:k // 3 + side:st, k % 3:k % 3 + side:st] += gt[..., k, :]
    return {"out": out, "gin": gin[:, 1:-1, 1:-1].contiguous(), "dw": dw.reshape(cout, 3, 3, cin),
            "db": g.sum((0, 1, 2))}


def _predict64(case, seed):
    """The network in 64 bits, with its BF16-rounded weights and inputs."""
    y, ys = _pairs(case, seed)
    x = []
    for t in (y.double(), ys.double()):
        m = t.mean((1, 2), keepdim=True)
        x.append((t - m) / (t.std((1, 2), correction=0, keepdim=True) + 1e-3))
    x = torch.stack(x, -1).bfloat16().double()
    g = torch.Generator(device="cpu").manual_seed(int(seed) % (1 << 31))
    for cin, cout, st, _ in LAYERS:
        w = torch.randn(cout * 9 * cin, generator=g) * math.sqrt(2.0 / (9 * cin))
        x = _conv64(x, w.bfloat16().reshape(cout, -1).to(_gpu()), torch.zeros(cout, device=_gpu()), st)
    n = x[0].numel()
    wfc = (torch.randn(n * 6, generator=g) * math.sqrt(1.0 / n)).to(_gpu()).double()
    return x.reshape(case["batch"], -1) @ wfc.reshape(n, 6)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("superpixel", "register"):
        return None  # clustering and the optimiser's accept / reject steps are discrete
    if kind == "layer":
        return _layer64(case, seed)
    if kind == "predict":
        return _predict64(case, seed)
    if kind == "batch":
        probs = _batch_problems(case, seed)
        if sum(int(p.patches.n_samples) for p in probs) > 12_000_000:
            return None
        parts = []
        for p in probs:
            X, y, state = p.volume().double(), p.observe(), None
            for _ in range(3):
                out, state = _sr64(p, X, y, "gauss", state)
                X = out["X"]
            parts.append(out)
        return {k: torch.cat([o[k] for o in parts]) for k in ("X", "e", "p", "W", "num", "den")}
    if _sizes(case["nx"], case["ny"], case["nz"], case["slices"], case["a"], case["stacks"])[0] \
            > 16_000_000:
        return None
    prob = _problem(case, seed)
    X = prob.volume().double()
    psf = case.get("psf", "gauss")
    if kind == "grad":
        N = prob.patches.n_samples
        dt = torch.float64 if case["f64"] else torch.float32
        gy = torch.randn(N, generator=_gen(seed * 7 + 9), device=_gpu()).to(dt).double()
        return _grad64(prob, X, gy)
    y = prob.observe()
    if kind == "forward":
        ys, valid = _forward64(prob, X, psf)
        return torch.where(valid, y.double() - ys, 0.0)
    if kind == "rebuild":
        one = torch.ones(prob.patches.n_samples, dtype=torch.float64, device=_gpu())
        num, den = _adjoint64(prob, y.double(), one, psf)
        return {"X0": _update64(prob, torch.zeros_like(X), num, den, lam=0.0, clamp=False),
                "num": num, "den": den}
    return _sr64(prob, X, y, psf)[0]
