"""Performance cases of the framework's public calls: what they are, how their
inputs are made, one pass of each, the work a pass cannot do without, and the
same result in 64 bits from plain torch.

A case is a dict of plain values; `kind` names the call it stands for:

  signatures  araullo_signatures on a specimen (ROI query, histograms, spectra)
  batch       the same as a stream of batches runs it: ar_roi_gather into kept
              buffers, then a tuned SignaturePlan replayed on them
  typed       araullo_signatures_typed, one channel per sub-lattice
  gather      ar_roi_gather alone, into kept buffers
  index       index_orientations against a library of rotated references
  sparse      index_orientations_sparse against its look-up table
  score       the structure-factor score through torch.autograd, forward and
              backward
  refine      refine.refine, descent steps on that score
  grid        ar_fsp_amplitudes on a cubic reciprocal-space grid

Sizes are those of the benchmark, its legs and the tests (R = 1 nm, 256 bins,
642 directions; R = 2 nm, 1024 bins, 10242 directions; 20000 and 100000
references; L = 64) and sizes around them.  All arrays are float32 except
orientations (float64) and indices: the interface has no other types.
"""
import math

import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import refine, synth

DEV = torch.device("cuda", 0)
A_AL, A_FE = 0.405, 0.287
F_AL = (4.2767, 4.9383, 6.9838, 8.1892)   # 1/d of fcc Al {111}, {200}, {220}, {311}, nm^-1
F_FE = (4.9276, 6.9686, 8.5347, 9.8552)   # 1/d of bcc Fe {110}, {200}, {211}, {220}, nm^-1
FCC = ((0.0, 0.0, 0.0), (0.0, 0.5, 0.5), (0.5, 0.0, 0.5), (0.5, 0.5, 0.0))
BCC = ((0.0, 0.0, 0.0), (0.5, 0.5, 0.5))
FAMILIES = (((1, 1, 1), (1, 0, 0), (1, 1, 0), (3, 1, 1)), ((1, 1, 0), (1, 0, 0), (2, 1, 1), (1, 1, 0)))
K_MAX = 10.0
MASKS = (0b11, 0b01, 0b10)                # every atom, the majority, the minority sub-lattice


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # a user trying one ROI interactively: latency and launches only
        {"name": "one_roi_signature", "kind": "signatures", "specimen": "grain", "n_roi": 1, "n_dir": 642,
         "nbins": 256, "radius": 1.0, "eta": 0.5},
        # a one-off call on a block of a specimen at the benchmark's resolution
        {"name": "box_signatures", "kind": "signatures", "specimen": "grain", "n_roi": 200, "n_dir": 10242,
         "nbins": 1024, "radius": 2.0, "eta": 0.5},
        # batches of a polycrystal, ROIs clipped at the surface, the plan and its buffers kept
        {"name": "clipped_batch", "kind": "batch", "specimen": "cone", "n_roi": 500, "n_dir": 10242, "nbins": 1024,
         "radius": 2.0, "eta": 0.5},
        # sub-lattice signatures of an ordered precipitate
        {"name": "sublattice_signatures", "kind": "typed", "specimen": "grain", "n_roi": 64, "n_dir": 2562,
         "nbins": 512, "radius": 1.5, "eta": 0.5},
        # the ROI query alone over a whole tip
        {"name": "tip_gather", "kind": "gather", "specimen": "cone", "n_roi": 8000, "radius": 2.0, "eta": 0.5},
        # a few ROIs against a coarse library
        {"name": "small_index", "kind": "index", "n_roi": 16, "n_lib": 1000, "n_dir": 642, "k": 1},
        # the benchmark's indexing stage
        {"name": "box_index", "kind": "index", "n_roi": 2000, "n_lib": 20000, "n_dir": 10242, "k": 16},
        # the two-phase leg: the largest batch the benchmark indexes
        {"name": "two_phase_index", "kind": "index", "n_roi": 20000, "n_lib": 100000, "n_dir": 10242, "k": 16},
        # the paper's sparse form on the benchmark's shape
        {"name": "box_sparse", "kind": "sparse", "n_roi": 2000, "n_lib": 20000, "n_dir": 10242, "n_hat": 1000,
         "k": 16},
        # the score and its gradient in a user's own optimiser
        {"name": "score_gradient", "kind": "score", "n_roi": 256, "n_dir": 10242, "n_freq": 4, "radius": 2.0},
        # a few descent steps of the refinement stage
        {"name": "refine_steps", "kind": "refine", "n_roi": 128, "n_dir": 10242, "n_freq": 4, "radius": 2.0,
         "steps": 6},
        # the paper's reciprocal-space benchmark, fewer ROIs
        {"name": "reciprocal_grid", "kind": "grid", "n_roi": 256, "L": 64, "radius": 2.0, "eta": 1.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mesh(rng, most=10242):
    """An icosphere of the levels in use, or a mesh of any size (odd ones too)."""
    if rng.random() < 0.6:
        return rng.choice([n for n in (162, 642, 2562, 10242) if n <= most])
    return _log_int(rng, 100, most)


def draw(rng):
    kind = rng.choice(["signatures", "batch", "typed", "gather", "index", "index", "sparse", "score", "refine",
                       "grid"])
    specimen = rng.choice(["grain", "cone"])
    radius = round(rng.uniform(0.8, 2.5), 2)
    eta = round(rng.uniform(0.3, 0.8), 2)
    if kind in ("signatures", "batch"):
        return {"kind": kind, "specimen": specimen, "n_roi": _log_int(rng, 1, 400), "n_dir": _mesh(rng),
                "nbins": rng.choice([256, 512, 1024, 1024, 2048]), "radius": radius, "eta": eta}
    if kind == "typed":
        return {"kind": kind, "specimen": "grain", "n_roi": _log_int(rng, 1, 100), "n_dir": _mesh(rng, 2562),
                "nbins": rng.choice([256, 512, 1024]), "radius": radius, "eta": eta}
    if kind == "gather":
        return {"kind": kind, "specimen": specimen, "n_roi": _log_int(rng, 1, 12000), "radius": radius, "eta": eta}
    if kind == "index":
        return {"kind": kind, "n_roi": _log_int(rng, 1, 5000), "n_lib": _log_int(rng, 200, 50000),
                "n_dir": _mesh(rng), "k": rng.choice([1, 5, 16, 16, 32, 64])}
    if kind == "sparse":
        return {"kind": kind, "n_roi": _log_int(rng, 1, 3000), "n_lib": _log_int(rng, 500, 20000),
                "n_dir": _mesh(rng), "n_hat": rng.randrange(100, 1200), "k": rng.choice([1, 16, 32])}
    if kind == "score":
        return {"kind": kind, "n_roi": _log_int(rng, 1, 300), "n_dir": _mesh(rng), "n_freq": rng.choice([1, 2, 4, 6]),
                "radius": radius}
    if kind == "refine":
        return {"kind": kind, "n_roi": _log_int(rng, 1, 100), "n_dir": _mesh(rng), "n_freq": rng.choice([2, 4]),
                "radius": radius, "steps": rng.randrange(2, 7)}
    return {"kind": kind, "n_roi": _log_int(rng, 1, 200), "L": rng.choice([32, 64, 64, 96]), "radius": radius,
            "eta": round(rng.uniform(0.5, 1.0), 2)}


# --------------------------------------------------------------------- inputs
def _gen(seed, stream):
    return torch.Generator(device=DEV).manual_seed(1000003 * int(seed) + stream)


def _uniform(gen, *shape):
    return torch.rand(shape, generator=gen, device=DEV, dtype=torch.float64)


def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float64)


def _directions(n):
    for level in range(7):
        if n == 10 * 4 ** level + 2:
            return torch.from_numpy(synth.icosphere(level)).to(DEV)
    i = torch.arange(n, dtype=torch.float64, device=DEV) + 0.5   # a golden spiral: any number of nodes
    z = 1.0 - 2.0 * i / n
    phi = math.pi * (1.0 + 5.0 ** 0.5) * i
    rho = torch.sqrt(1.0 - z * z)
    return torch.stack([rho * torch.cos(phi), rho * torch.sin(phi), z], 1).float().contiguous()


def _quats(gen, n):
    q = _normal(gen, n, 4)
    return (q / q.norm(dim=1, keepdim=True)).contiguous()


def _matrices(q):
    """[n][3][3] rotation matrices of quaternions (w, x, y, z)."""
    w, x, y, z = (q / q.norm(dim=-1, keepdim=True)).unbind(-1)
    m = [1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
         2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
         2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]
    return torch.stack(m, -1).reshape(*q.shape[:-1], 3, 3)


def _lattice(basis, a, q, lo, hi):
    """Sites (float64) of a rotated crystal inside the box, and each site's index in the basis."""
    lo, hi = (torch.tensor(v, dtype=torch.float64, device=DEV) for v in (lo, hi))
    half = int(math.ceil(float((hi - lo).norm()) / 2 / a)) + 1
    r = torch.arange(-half, half + 1, dtype=torch.float64, device=DEV)
    M = _matrices(q)
    sites, kinds = [], []
    for b, off in enumerate(basis):
        for part in r.split(32):
            p = torch.cartesian_prod(part, r, r) + torch.tensor(off, dtype=torch.float64, device=DEV)
            p = (p * a) @ M.T + (lo + hi) / 2
            p = p[((p >= lo) & (p < hi)).all(1)]
            sites.append(p)
            kinds.append(torch.full((len(p),), b, dtype=torch.int32, device=DEV))
    return torch.cat(sites), torch.cat(kinds)


def _thin(gen, pos, kinds, eta, sigma):
    """The detected fraction of the sites, in measured (shuffled) order, displaced."""
    keep = torch.randperm(len(pos), generator=gen, device=DEV)[:int(round(eta * len(pos)))]
    pos = pos[keep]
    return (pos + sigma * _normal(gen, *pos.shape)).float().contiguous(), kinds[keep].contiguous()


def _specimen(case, seed):
    """(positions, types, centres): a single grain around its ROIs, or a tip of several grains
    whose ROIs the surface clips."""
    gen, R = _gen(seed, 1), case["radius"]
    if case["specimen"] == "grain":
        n = max(1, math.ceil((case["n_roi"] / 2) ** (1 / 3)))
        box = (2.0 * n, 2.0 * n, 2.0 * math.ceil(case["n_roi"] / n ** 2))
        sites, kinds = _lattice(FCC, A_AL, _quats(gen, 1)[0], [-R] * 3, [v + R for v in box])
        pos, kinds = _thin(gen, sites, kinds, case["eta"], 0.05)
        centres = _uniform(gen, case["n_roi"], 3) * torch.tensor(box, dtype=torch.float64, device=DEV)
        return pos, (kinds == 0).to(torch.int32).contiguous(), centres.float().contiguous()
    height, top, bottom = 60.0, 15.0, 25.6
    seeds = _uniform(gen, 8, 3) * 2 - 1
    seeds = seeds * torch.tensor([bottom, bottom, height / 2], dtype=torch.float64, device=DEV)
    seeds[:, 2] += height / 2
    quats, parts = _quats(gen, 8), []
    for g in range(8):
        basis, a = ((FCC, A_AL), (BCC, A_FE))[g % 2]
        p, _ = _lattice(basis, a, quats[g], [-bottom, -bottom, 0.0], [bottom, bottom, height])
        p = p[p[:, :2].norm(dim=1) <= bottom + (top - bottom) * p[:, 2] / height]
        near = torch.stack([((p - s) ** 2).sum(1) for s in seeds], 1).argmin(1)
        parts.append(p[near == g])
    sites = torch.cat(parts)
    pos, kinds = _thin(gen, sites, torch.zeros(len(sites), dtype=torch.int32, device=DEV), case["eta"], 0.05)
    at = torch.randint(len(pos), (case["n_roi"],), generator=gen, device=DEV)
    centres = pos[at].double() + 0.5 * R * (2 * _uniform(gen, case["n_roi"], 3) - 1)
    return pos, kinds, centres.float().contiguous()


def _family(hkl):
    """One unit vector per antipodal pair of the cubic family {hkl}."""
    a, b, c = hkl
    seen, out = set(), []
    for p in {(a, b, c), (a, c, b), (b, a, c), (b, c, a), (c, a, b), (c, b, a)}:
        for s in range(8):
            v = tuple(x if (s >> i) & 1 == 0 or x == 0 else -x for i, x in enumerate(p))
            if v not in seen and tuple(-x for x in v) not in seen:
                seen.add(v)
                out.append(v)
    t = torch.tensor(sorted(out), dtype=torch.float64, device=DEV)
    return t / t.norm(dim=1, keepdim=True)


def _images(dirs, quats, phase, background, gen=None, noise=0.0, gain=1.0):
    """[n][4][n_dir] float32 window images of rotated crystals: peaks about 10 degrees wide along
    the plane normals over a background, `gain` the counts scale, noise relative."""
    d = dirs.float()
    out = torch.empty((len(quats), 4, len(d)), dtype=torch.float32, device=DEV)
    M = _matrices(quats).float()
    step = max(1, 40_000_000 // len(d))
    for ph in (0, 1):
        rows = (phase == ph).nonzero().flatten()
        for part in rows.split(step):
            for w in range(4):
                axes = _family(FAMILIES[ph][w]).float()
                img = torch.full((len(part), len(d)), background, dtype=torch.float32, device=DEV)
                for a in axes:
                    img += torch.exp(((M[part] @ a) @ d.T).abs_().sub_(1.0).div_(0.015))
                if noise:
                    img *= 1.0 + noise * torch.randn(img.shape, generator=gen, device=DEV)
                    img.clamp_(min=0.0)
                out[part, w] = img * gain
    return out


def _index_inputs(case, seed):
    """(library orientations, phases, reference images, ROI images): references of two phases, ROIs
    near library orientations under measured noise."""
    gen = _gen(seed, 2)
    dirs = _directions(case["n_dir"])
    n_lib, n_roi = case["n_lib"], case["n_roi"]
    quats = _quats(gen, n_lib)
    phase = (torch.arange(n_lib, device=DEV) >= (n_lib + 1) // 2).to(torch.int32)
    refs = _images(dirs, quats, phase, 0.1, gain=1000.0)
    at = torch.randint(n_lib, (n_roi,), generator=gen, device=DEV)
    q = quats[at] + 0.02 * _normal(gen, n_roi, 4)
    rois = _images(dirs, q / q.norm(dim=1, keepdim=True), phase[at], 0.25, gen, 0.25, 400.0)
    return quats, phase, refs, rois


def _sparse_inputs(case, seed):
    """(reference image, directions, library orientations, ROI images) of one phase."""
    gen = _gen(seed, 3)
    dirs = _directions(case["n_dir"])
    zero = torch.zeros(1, dtype=torch.int32, device=DEV)
    ident = torch.tensor([[1.0, 0.0, 0.0, 0.0]], dtype=torch.float64, device=DEV)
    ref = _images(dirs, ident, zero, 0.05, gen, 0.02, 1000.0)
    quats = _quats(gen, case["n_lib"])
    q = quats[torch.randint(case["n_lib"], (case["n_roi"],), generator=gen, device=DEV)]
    q = q + 0.02 * _normal(gen, *q.shape)
    rois = _images(dirs, q / q.norm(dim=1, keepdim=True), zero.expand(len(q)), 0.25, gen, 0.25, 400.0)
    return ref, dirs, quats, rois


def _balls(gen, n_roi, radius, eta, sigma):
    """CSR of ROIs cut from rotated crystals of two phases: (rel, offsets, orientations, phases)."""
    quats = _quats(gen, n_roi)
    phase = torch.randint(2, (n_roi,), generator=gen, device=DEV).to(torch.int32)
    M = _matrices(quats)
    rows = [None] * n_roi
    for ph, (basis, a) in enumerate(((FCC, A_AL), (BCC, A_FE))):
        half = int(math.ceil(radius / a)) + 2
        r = torch.arange(-half, half + 1, dtype=torch.float64, device=DEV)
        cells = torch.cartesian_prod(r, r, r)
        sites = torch.cat([cells + torch.tensor(o, dtype=torch.float64, device=DEV) for o in basis])
        for i in (phase == ph).nonzero().flatten().tolist():
            p = ((sites + _uniform(gen, 1, 3)) * a) @ M[i].T
            p = p[torch.rand(len(p), generator=gen, device=DEV) < eta]
            p = (p + sigma * _normal(gen, *p.shape)).float()
            rows[i] = p[(p * p).sum(1) <= radius * radius]
    rel = torch.zeros((sum(len(p) for p in rows), 4), dtype=torch.float32, device=DEV)
    rel[:, :3] = torch.cat(rows)
    offsets = torch.tensor([0] + [len(p) for p in rows], dtype=torch.int64, device=DEV).cumsum(0)
    return rel, offsets.contiguous(), quats, phase


def _score_inputs(case, seed):
    gen = _gen(seed, 4)
    rel, offsets, quats, phase = _balls(gen, case["n_roi"], case["radius"], 0.5, 0.05)
    dirs = _directions(case["n_dir"])
    nf = case["n_freq"]
    freqs = torch.tensor([(F_AL + F_FE)[:nf], (F_FE + F_AL)[:nf]], dtype=torch.float32, device=DEV)
    # targets: the amplitudes of one noise-free, unrotated crystal per phase
    targets = torch.empty((2, nf, len(dirs)), dtype=torch.float32, device=DEV)
    for ph, (basis, a) in enumerate(((FCC, A_AL), (BCC, A_FE))):
        half = int(math.ceil(case["radius"] / a)) + 1
        r = torch.arange(-half, half + 1, dtype=torch.float64, device=DEV)
        p = torch.cat([torch.cartesian_prod(r, r, r) + torch.tensor(o, dtype=torch.float64, device=DEV)
                       for o in basis]) * a
        p = p[(p * p).sum(1) <= case["radius"] ** 2]
        for w in range(nf):
            t = 2 * math.pi * float(freqs[ph, w]) * (dirs.double() @ p.T)
            targets[ph, w] = (torch.complex(t.cos().sum(1), t.sin().sum(1)).abs() / len(p)).float()
    q = quats + 0.01 * _normal(gen, *quats.shape)        # about a degree off, as a library's best entry is
    return {"rel": rel, "offsets": offsets, "quats": (q / q.norm(dim=1, keepdim=True)).float().contiguous(),
            "phase": phase, "dirs": dirs, "freqs": freqs, "targets": targets}


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case, "ctx": nat.Context(0)}
    if kind in ("signatures", "batch", "typed", "gather"):
        state["pos"], state["types"], state["centres"] = _specimen(case, seed)
        if kind == "gather":
            # room for complete ROIs of the denser phase
            rows = case["n_roi"] * int(90.0 * case["eta"] * 4.19 * case["radius"] ** 3 + 200)
            state["off"] = torch.zeros(case["n_roi"] + 1, dtype=torch.int64, device=DEV)
            state["rel"] = torch.zeros((rows, 4), device=DEV)
            return state
        state["dirs"] = _directions(case["n_dir"])
        state["windows"] = nat.windows_for(case["radius"], case["nbins"], synth.window_spacings())
        if kind == "batch":
            off, rel = nat.ar_roi_gather(state["ctx"], state["pos"], state["centres"], case["radius"])
            n_roi, n_win = case["n_roi"], len(state["windows"])
            state["off"], state["rel"] = off, torch.empty((len(rel) + len(rel) // 20 + 64, 4), device=DEV)
            state["images"] = torch.empty((n_roi, n_win, case["n_dir"]), device=DEV)
            state["plan"] = nat.SignaturePlan(state["ctx"], n_roi, len(state["rel"]), case["n_dir"], case["nbins"],
                                              n_win)
            state["plan"].tune(rel, off, case["radius"], state["dirs"], state["windows"], out=state["images"])
    elif kind == "index":
        state["quats"], state["phase"], state["refs"], state["rois"] = _index_inputs(case, seed)
        state["lib"] = nat.Library(state["ctx"], state["refs"], state["quats"], state["phase"])
    elif kind == "sparse":
        ref, dirs, quats, state["rois"] = _sparse_inputs(case, seed)
        state["lut"] = nat.SparseLUT(state["ctx"], ref, dirs, quats, [case["n_lib"]],
                                     min(case["n_hat"], 4 * case["n_dir"]))
    elif kind in ("score", "refine"):
        state.update(_score_inputs(case, seed))
    else:
        gen = _gen(seed, 5)
        state["rel"], state["offsets"], _, _ = _balls(gen, case["n_roi"], case["radius"], case["eta"], 0.0)
    return state


# ----------------------------------------------------------------------- pass
def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "signatures":
        return nat.araullo_signatures(ctx, state["pos"], state["centres"], case["radius"], state["dirs"],
                                      case["nbins"], state["windows"])
    if kind == "batch":
        off, rel = nat.ar_roi_gather(ctx, state["pos"], state["centres"], case["radius"],
                                     out=(state["off"], state["rel"]))
        return state["plan"].run(rel, off, case["radius"], state["dirs"], state["windows"], out=state["images"])
    if kind == "typed":
        return nat.araullo_signatures_typed(ctx, state["pos"], state["types"], state["centres"], case["radius"],
                                            state["dirs"], case["nbins"], state["windows"], MASKS)
    if kind == "gather":
        nat.ar_roi_gather(ctx, state["pos"], state["centres"], case["radius"], out=(state["off"], state["rel"]))
        return state["off"], state["rel"]
    if kind == "index":
        return nat.index_orientations(ctx, state["rois"], state["lib"], case["k"])
    if kind == "sparse":
        return nat.index_orientations_sparse(ctx, state["rois"], state["lut"], case["k"])
    if kind == "score":
        q = state["quats"].clone().requires_grad_(True)
        score = refine.sf_score(ctx, q, state["rel"], state["offsets"], state["phase"], state["dirs"],
                                state["freqs"], state["targets"])
        score.sum().backward()
        return score.detach(), q.grad
    if kind == "refine":
        q = state["quats"].clone()
        score = refine.refine(ctx, q, state["rel"], state["offsets"], state["phase"], state["dirs"], state["freqs"],
                              state["targets"], steps=case["steps"], a0=0.01)
        return q, score
    return nat.ar_fsp_amplitudes(ctx, state["rel"], state["offsets"], case["L"], K_MAX)


# ----------------------------------------------------------------------- work
def _atoms_per_roi(case):
    """Atoms of a complete ROI (60 sites per nm^3 in fcc Al), two thirds of it where a surface clips."""
    full = 60.2 * case.get("eta", 0.5) * 4.19 * case["radius"] ** 3
    return full * (0.67 if case.get("specimen") == "cone" else 1.0)


def _specimen_atoms(case):
    if case["specimen"] == "cone":
        return 60.2 * case["eta"] * math.pi * 60.0 * (15.0 ** 2 + 15.0 * 25.6 + 25.6 ** 2) / 3.0
    n, R = max(1, math.ceil((case["n_roi"] / 2) ** (1 / 3))), case["radius"]
    return 60.2 * case["eta"] * (2 * n + 2 * R) ** 2 * (2 * math.ceil(case["n_roi"] / n ** 2) + 2 * R)


def work(case):
    """Inputs read once, outputs written once; arithmetic as the method counts it: 7 flops per
    projected atom and 2.5 N log2 N per real transform, 2 per multiply-add of Eq. S1, 18.25 per
    term of the score with its gradient and 6.25 without, 8 per complex multiply-add of Eq. (2)."""
    kind, n_roi = case["kind"], case["n_roi"]
    if kind in ("signatures", "batch", "typed", "gather"):
        nbytes = 12.0 * _specimen_atoms(case) + 12.0 * n_roi
        gathered = n_roi * _atoms_per_roi(case)
        if kind == "gather":
            return {"bytes": nbytes + 16.0 * gathered + 8.0 * n_roi, "flops": 8.0 * gathered}
        ch = len(MASKS) if kind == "typed" else 1
        nb = case["nbins"]
        share = 2.0 if kind == "typed" else 1.0    # every atom, and once more over the two sub-lattices
        flops = case["n_dir"] * (7.0 * gathered * share + ch * n_roi * 2.5 * nb * math.log2(nb))
        return {"bytes": nbytes + 12.0 * case["n_dir"] + ch * 16.0 * n_roi * case["n_dir"], "flops": flops}
    if kind == "index":
        K, n_lib = 4.0 * case["n_dir"], case["n_lib"]
        return {"bytes": 4.0 * K * n_roi + 2.0 * K * n_lib + 8.0 * case["k"] * n_roi,
                "flops": 2.0 * n_roi * n_lib * K}
    if kind == "sparse":
        terms = float(n_roi) * case["n_lib"] * case["n_hat"]
        return {"bytes": 16.0 * case["n_dir"] * n_roi + 2.0 * case["n_lib"] * case["n_hat"] + 8.0 * case["k"] * n_roi,
                "flops": 3.0 * terms}
    atoms = n_roi * _atoms_per_roi(case)
    if kind in ("score", "refine"):
        terms = atoms * case["n_freq"] * case["n_dir"] / 2.0    # antipodal directions share a term
        grads = 1 if kind == "score" else case["steps"]
        nbytes = 16.0 * atoms + 8.0 * (1 + case["n_freq"]) * case["n_dir"] + 40.0 * n_roi
        return {"bytes": nbytes * (grads + 1), "flops": terms * (18.25 * grads + 6.25)}
    return {"bytes": 16.0 * atoms + 4.0 * n_roi * case["L"] ** 3, "flops": 8.0 * atoms * case["L"] ** 3}


# ---------------------------------------------------------------- in 64 bits
def _windows64(case):
    """Bins k = L / d of each spacing interval, L = 2R + 2dR."""
    R, nb = case["radius"], case["nbins"]
    span = 2 * R + 2 * R / (nb // 2 - 1)
    return [(math.ceil(span / hi), math.floor(span / lo)) for lo, hi in synth.window_spacings().tolist()]


def _inside(pos, centre, radius):
    """Relative coordinates of a ROI's atoms: membership and coordinates are defined in FP32."""
    d = pos - centre
    dd = d.double()
    s = (dd[:, 0] * dd[:, 0]).float().double()
    s = (dd[:, 1] * dd[:, 1] + s).float().double()
    s = (dd[:, 2] * dd[:, 2] + s).float()
    near = s <= float(torch.tensor(radius, dtype=torch.float32).double() ** 2)
    return d[near], near


def _exact_images(case, pos, select, centres, dirs):
    """Window maxima of the spectra of the Eq. (1) histograms (whose bin of an atom is defined in
    FP32), the transform in 64 bits: [n_roi][n_win][n_dir] and the counts."""
    nb, wins = case["nbins"], _windows64(case)
    R = float(torch.tensor(case["radius"], dtype=torch.float32))
    dR = R / (nb // 2 - 1)
    shift = torch.tensor(R + dR, dtype=torch.float64).float().to(DEV)
    scale = torch.tensor(nb / (2 * R + 2 * dR), dtype=torch.float64).float().to(DEV)
    lo, hi = min(w[0] for w in wins), max(w[1] for w in wins)
    k = torch.arange(lo, hi + 1, dtype=torch.float64, device=DEV)
    n = torch.arange(nb, dtype=torch.float64, device=DEV)
    turn = 2 * math.pi * ((n[:, None] * k[None]) % nb) / nb
    C, S = turn.cos(), turn.sin()
    out = torch.zeros((len(centres), len(wins), len(dirs)), dtype=torch.float64, device=DEV)
    count = torch.zeros(len(centres), dtype=torch.int64, device=DEV)
    v = dirs.double()
    for r, c in enumerate(centres):
        x, near = _inside(pos, c, R)
        if select is not None:
            x = x[select[near]]
        count[r] = len(x)
        if not len(x):
            continue
        xd = x.double()
        s = (v[:, 0:1] * xd[:, 0]).float().double()
        s = (v[:, 1:2] * xd[:, 1] + s).float().double()
        s = (v[:, 2:3] * xd[:, 2] + s).float()
        b = ((s + shift) * scale).clamp_(0, nb - 1).long()
        hist = torch.zeros((len(v), nb), dtype=torch.float64, device=DEV)
        hist.scatter_add_(1, b, torch.ones(1, dtype=torch.float64, device=DEV).expand(b.shape))
        amp = torch.hypot(hist @ C, hist @ S)
        for w, (a, z) in enumerate(wins):
            out[r, w] = amp[:, a - lo:z - lo + 1].amax(1)
    return out, count


def _normalised64(img):
    top = img.double().amax(2, keepdim=True)
    return torch.where(top > 0, img.double() / top, torch.zeros((), dtype=torch.float64, device=DEV)).flatten(1)


def _exact_index(case, seed):
    _, _, refs, rois = _index_inputs(case, seed)
    S = _normalised64(rois)
    n2 = (S * S).sum(1, keepdim=True)
    best = torch.full((len(S), case["k"]), math.inf, dtype=torch.float64, device=DEV)
    for part in refs.split(max(1, 400_000_000 // S.shape[1])):
        L = _normalised64(part)
        d = (n2 + (L * L).sum(1)[None] - 2 * (S @ L.T)).clamp_(min=0)
        best = torch.cat([best, d], 1).topk(case["k"], dim=1, largest=False).values
    return [None, best]


def _exact_sparse(case, seed):
    ref, dirs, quats, rois = _sparse_inputs(case, seed)
    n_dir, n_hat = case["n_dir"], min(case["n_hat"], 4 * case["n_dir"])
    key = _normalised64(ref)[0]
    order = torch.sort(key, descending=True, stable=True).indices[:n_hat]
    val, win, node = key[order].float().double(), order // n_dir, order % n_dir
    S = _normalised64(rois).reshape(len(rois), 4, n_dir).permute(1, 2, 0).reshape(4 * n_dir, len(rois)).contiguous()
    v, M = dirs.double(), _matrices(quats)
    best = torch.full((len(rois), case["k"]), math.inf, dtype=torch.float64, device=DEV)
    step = max(1, int(200_000_000 // (n_hat * max(len(rois), n_dir))))
    for part in M.split(step):
        u = (part @ v[node].T).transpose(1, 2)                   # [g][i][3]
        p = torch.cat([(x @ v.T).argmax(1, keepdim=True).T for x in u])
        d = ((S[(win * n_dir)[None] + p] - val[None, :, None]) ** 2).sum(1).T
        best = torch.cat([best, d], 1).topk(case["k"], dim=1, largest=False).values
    return [None, best]


def _score64(s, r, q, grad):
    """J of ROI r at quaternion q (float64) and, if asked, dJ/dq."""
    a, z = int(s["offsets"][r]), int(s["offsets"][r + 1])
    x, n, ph = s["rel"][a:z, :3].double(), s["dirs"].double(), int(s["phase"][r])
    q = q.detach().clone().requires_grad_(grad)
    M = _matrices(q)
    u = n @ M.detach().T
    t = u @ x.T
    J, du = torch.zeros((), dtype=torch.float64, device=DEV), torch.zeros_like(u)
    for w in range(s["freqs"].shape[1]):
        f = float(s["freqs"][ph, w])
        th = 2 * math.pi * f * t
        c, sn = th.cos(), th.sin()
        C, S = c.sum(1), sn.sum(1)
        mag = torch.hypot(C, S)
        e = mag / len(x) - s["targets"][ph, w].double()
        J = J + (e * e).sum()
        if grad:
            k = torch.where(mag >= 1e-12 * len(x), 4 * math.pi * f * e / (len(x) * mag), torch.zeros_like(mag))
            du += k[:, None] * (S[:, None] * (c @ x) - C[:, None] * (sn @ x))
    if not grad:
        return J, None
    return J, torch.autograd.grad(M, q, grad_outputs=du.T @ n)[0]


def _exact_refine(case, seed):
    s = _score_inputs(case, seed)
    qs, Js = [], []
    for r in range(case["n_roi"]):
        q, a = s["quats"][r].double(), 0.01
        J, g = _score64(s, r, q, True)
        for it in range(case["steps"]):
            t = q - a * g / g.norm()
            t = t / t.norm()
            Jt, gt = _score64(s, r, t, it + 1 < case["steps"])
            if float(Jt) <= float(J) - 1e-4 * a * float(g.norm()):
                q, J, g, a = t, Jt, gt if gt is not None else g, 1.5 * a
            else:
                a *= 0.5
        qs.append(q)
        Js.append(J)
    return torch.stack(qs), torch.stack(Js)


def _exact_grid(case, seed):
    rel, offsets, _, _ = _balls(_gen(seed, 5), case["n_roi"], case["radius"], case["eta"], 0.0)
    L = case["L"]
    k = (torch.arange(L, dtype=torch.float64, device=DEV) - L // 2) * (2 * K_MAX / L)
    out = torch.empty((case["n_roi"], L, L, L), dtype=torch.float64, device=DEV)
    for r in range(case["n_roi"]):
        x = rel[offsets[r]:offsets[r + 1], :3].double()
        X, Y, Z = (torch.polar(torch.ones((), dtype=torch.float64, device=DEV), -2 * math.pi * k[:, None] * x[:, a])
                   for a in range(3))
        for b in range(0, L, 32):
            B = (Y[b:b + 32, None] * Z[None]).reshape(-1, len(x))
            out[r, :, b:b + 32] = (X @ B.T).abs().reshape(L, -1, L)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("signatures", "batch", "typed"):
        pos, types, centres = _specimen(case, seed)
        dirs = _directions(case["n_dir"])
        if kind == "typed":
            per = [_exact_images(case, pos, ((m >> types.long()) & 1).bool(), centres, dirs)[0] for m in MASKS]
            return [torch.stack(per, 1), None]
        img, _ = _exact_images(case, pos, None, centres, dirs)
        return img if kind == "batch" else [img, None]
    if kind == "index":
        return _exact_index(case, seed)
    if kind == "sparse":
        return _exact_sparse(case, seed)
    if kind == "score":
        s = _score_inputs(case, seed)
        both = [_score64(s, r, s["quats"][r].double(), True) for r in range(case["n_roi"])]
        return torch.stack([J for J, _ in both]).detach(), torch.stack([g for _, g in both])
    if kind == "refine":
        return _exact_refine(case, seed)
    if kind == "grid":
        return _exact_grid(case, seed)
    return None          # the gathered rows are FP32 differences, bit for bit
