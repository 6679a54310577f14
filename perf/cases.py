"""Performance cases of the alignment library: what a program asks of it, from
one particle against a resident reference set to tens of thousands.

``listed()`` gives the fixed cases, ``draw(rng)`` one more of the same ranges,
``prepare`` what the program holds before the call (a context, resident
references, particle stacks on the GPU), ``run`` one pass through the public
entry points, ``work`` the arithmetic and bytes that the pass cannot do
without, ``exact`` the same results in 64 bits from plain torch.

Particles are rendered blob references with a random rotation, shift and
mirror at SNR 0.05 or 0.1, as in the repository's benchmark workloads.
"""

from __future__ import annotations

import math

import torch

from paper_2011_05755_amd import mra, synth

NPHI = 256
BIG = 64 << 30  # workspace of a program that has most of the GPU to itself


def listed():
    return [
        # One new particle against a resident reference set: the smallest call,
        # as made by a program that aligns images as they come off the detector.
        dict(name="one_particle_fp32", kind="align", prec="fp32", N=1, L=76, K=100, T=3, r_max=35, snr=0.05),
        # A tight serving loop that may not allocate: a dozen small boxes a call.
        dict(name="serve_noalloc_bf16", kind="noalloc", prec="bf16", N=12, L=64, K=20, T=2, r_max=30, snr=0.1),
        # Iterative 2-D classification of the 1000-particle workload: three passes
        # of new references, alignment and average update.
        dict(name="small_classify_fp32", kind="classify", prec="fp32", N=1000, L=64, K=10, T=2, r_max=30, snr=0.1,
             iters=3),
        # The throughput workload's shapes (76 px, 100 references, +-3 px), a
        # tenth and a fifth of its particles: the work of every pass of a
        # 2-D classification, in full precision and on 16-bit matrix cores.
        dict(name="stack_76px_fp32", kind="align", prec="fp32", N=10000, L=76, K=100, T=3, r_max=35, snr=0.05),
        dict(name="stack_76px_bf16", kind="align", prec="bf16", N=20000, L=76, K=100, T=3, r_max=35, snr=0.05),
        # The paper's 90 px particles in FP16, with the sub-step angle that a
        # refinement that follows takes as its start.
        dict(name="stack_90px_fp16_angle", kind="align", prec="fp16", N=3001, L=90, K=50, T=3, r_max=36, snr=0.05,
             psi_frac=True),
        # Medium boxes with the runner-up, from which a program judges how sure
        # an assignment is; an odd number of references.
        dict(name="stack_96px_fp32_cc2", kind="align", prec="fp32", N=700, L=96, K=61, T=2, r_max=46, snr=0.05,
             cc2=True),
        # Large boxes of the uneven production load: many references, many rings.
        dict(name="large_128px_bf16", kind="align", prec="bf16", N=1200, L=128, K=200, T=4, r_max=62, snr=0.05),
        # Several requests of uneven size in one batched call (the server's step).
        dict(name="batch_uneven_bf16", kind="batch", prec="bf16", N=1500, L=76, K=60, T=3, r_max=35, snr=0.05,
             stacks=5),
        # New references, then a short stack against them: the first step of
        # every outer iteration, and of a server that takes a new model.
        dict(name="new_refs_fp32", kind="reload", prec="fp32", N=64, L=90, K=100, T=2, r_max=36, snr=0.1),
        # Reference-free alignment of one class: three passes from the mean.
        dict(name="rfa_loop", kind="rfa", prec="fp32", N=8000, L=76, K=1, T=3, r_max=35, snr=0.05, iters=3),
        # The class-average update of a full classification pass.
        dict(name="class_averages", kind="averages", prec="fp32", N=50000, L=76, K=100, T=3, r_max=35, snr=0.05),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["align"] * 6 + ["noalloc", "batch", "reload", "classify", "rfa", "averages"])
    L = rng.choice([64, 76, 90, 96, 128, 65, 83, 101])
    T = rng.choice([1, 2, 3, 3, 4, 5])
    c = dict(kind=kind, prec=rng.choice(["fp32", "bf16", "fp16"]), L=L, T=T, r_max=rng.randint(L // 3, L // 2 - 2),
             snr=rng.choice([0.05, 0.1]))
    if kind == "rfa":
        c.update(prec="fp32", K=1, N=_log(rng, 100, 6000), iters=rng.randint(2, 4))
        return c
    c["K"] = _log(rng, 5, 300)
    if kind == "averages":
        c.update(prec="fp32", N=_log(rng, 500, 50000))
        c["N"] = min(c["N"], 50000 * 76 * 76 // (L * L))
        return c
    # at most half the arithmetic of the largest listed case, a third of that in
    # FP32 with its slower matrix cores
    room = 0.5 * 20000 * 49 * 100 * 35 * (0.33 if c["prec"] == "fp32" else 1.0)
    most = int(room / ((2 * T + 1) ** 2 * c["K"] * c["r_max"]))
    if kind == "align":
        c["N"] = _log(rng, 1, max(2, min(most, 20000)))
        if rng.random() < 0.25:
            c["cc2"] = True
        if rng.random() < 0.25:
            c["psi_frac"] = True
    elif kind == "noalloc":
        c["N"] = _log(rng, 1, max(2, min(most, 200)))
    elif kind == "reload":
        c["N"] = _log(rng, 8, max(9, min(most, 500)))
    elif kind == "classify":
        c["iters"] = rng.randint(2, 3)
        c["N"] = _log(rng, 200, max(201, min(most // 3, 3000)))
    else:
        c["stacks"] = rng.randint(2, 8)
        c["N"] = _log(rng, 20, max(21, min(most // c["stacks"], 2000)))
    return c


def _stacks(case):
    """(N, L, K, T, r_max) of every stack of a case: one, but for a batch, whose
    stacks differ in size, box, references and search range."""
    base = (case["N"], case["L"], case["K"], case["T"], case["r_max"])
    out = [base]
    for i in range(1, case.get("stacks", 1)):
        N, L, K, T, r = base
        L2 = L - 12 * (i % 2)
        out.append((max(1, N * (1 + i % 3) // (2 + i)), L2, max(2, K - 7 * i if K > 7 * i + 2 else K), max(1, T - i % 2),
                    min(r, L2 // 2 - 2)))
    return out


def _inputs(case, seed, device):
    """Reference images and particles of every stack, from the seed alone."""
    got = []
    for i, (N, L, K, T, r_max) in enumerate(_stacks(case)):
        blobs = synth.make_blobs(K, L, seed=(seed, 2 * i), rho_max=min(L / 2 - 4, r_max + 1.0))
        refs = synth.render_refs(blobs, device=device)
        parts, truth = synth.make_particles(blobs, N, T, case["snr"], seed=(seed, 2 * i + 1), n_phi_grid=None,
                                            device=device)
        got.append((refs, parts, truth))
    return got


def _load(ctx, rid, refs, case, T, r_max):
    ctx.load_refs(rid, refs, r_min=1, r_max=r_max, shift_max=T, precision=case["prec"])


def prepare(case, seed):
    dev = torch.device("cuda", 0)
    data = _inputs(case, seed, dev)
    ctx = mra.Context(0, workspace_cap=BIG if case["N"] >= 1000 else 0)
    state = dict(case=case, ctx=ctx, data=data)
    shapes = _stacks(case)
    if case["kind"] == "averages":
        refs, parts, truth = data[0]
        i32 = dict(dtype=torch.int32, device=dev)
        psi = (truth.alpha * (NPHI / (2 * math.pi))).round().astype("int64") % NPHI
        p = mra.AlignResult.empty(case["N"], dev)
        for t, v in ((p.ref, truth.ref), (p.shift_x, truth.shift_x), (p.shift_y, truth.shift_y), (p.psi, psi),
                     (p.mirror, truth.mirror)):
            t.copy_(torch.as_tensor(v).to(**i32))
        state.update(params=p, averages=refs.clone())
    if case["kind"] not in ("reload", "rfa", "classify"):
        for i, (refs, _, _) in enumerate(data):
            _load(ctx, i, refs, case, shapes[i][3], shapes[i][4])
    if case["kind"] in ("noalloc", "batch"):
        state["outs"] = [mra.AlignResult.empty(s[0], dev) for s in shapes]
    return state


def _fields(r):
    return {k: getattr(r, k) for k in ("ref", "shift_x", "shift_y", "psi", "mirror", "cc", "cc2", "flat_index",
                                       "psi_frac") if getattr(r, k) is not None}


def run(state):
    case, ctx, data = state["case"], state["ctx"], state["data"]
    kind, (refs, parts, _) = case["kind"], data[0]
    if kind == "align":
        return _fields(ctx.align(0, parts, with_cc2=case.get("cc2", False), with_psi_frac=case.get("psi_frac", False)))
    if kind == "noalloc":
        return _fields(ctx.align_noalloc(0, parts, state["outs"][0]))
    if kind == "batch":
        ctx.align_batch([(i, d[1], -1, o) for i, (d, o) in enumerate(zip(data, state["outs"]))])
        return [_fields(o) for o in state["outs"]]
    if kind == "reload":
        _load(ctx, 0, refs, case, case["T"], case["r_max"])
        return _fields(ctx.align(0, parts))
    if kind == "rfa":
        out, avg, passes, changed = ctx.rfa(0, parts, r_min=1, r_max=case["r_max"], shift_max=case["T"],
                                            max_iter=case["iters"])
        return dict(_fields(out), average=avg, passes=passes)
    if kind == "classify":
        averages = refs.clone()
        out, counts, passes, changed = ctx.classify(0, parts, averages, r_min=1, r_max=case["r_max"],
                                                    shift_max=case["T"], max_iter=case["iters"],
                                                    max_changed_frac=0.0, precision=case["prec"])
        return dict(_fields(out), averages=averages, counts=counts, passes=passes)
    counts = ctx.update_averages(0, parts, state["params"], state["averages"])
    return dict(averages=state["averages"], counts=counts)


def work(case):
    """Each image and reference read once, each result written once; per
    particle and shift the bilinear samples (8 operations each) and the real
    FFT of every ring; per shift and reference the ring correlation of both
    mirrors (1024 per ring: 4 real products over 128 frequencies)."""
    nbytes = flops = 0.0
    for N, L, K, T, r_max in _stacks(case):
        S = (2 * T + 1) ** 2
        if case["kind"] == "averages":
            nbytes += 4.0 * L * L * (N + 2 * K) + 20.0 * N + 4.0 * K
            flops += 24.0 * L * L * N
            continue
        passes = case.get("iters", 1)
        nbytes += passes * (4.0 * L * L * (N + K) + 28.0 * N)
        per_row = r_max * (NPHI * 8 + 2.5 * NPHI * math.log2(NPHI))
        flops += passes * N * S * (per_row + K * 1024.0 * r_max)
        if case["kind"] in ("rfa", "classify"):
            flops += passes * 24.0 * L * L * N
    return dict(bytes=nbytes, flops=flops)


# ---- the same results in 64 bits, from plain torch ----

def _angles(dev):
    return 2.0 * math.pi * torch.arange(NPHI, dtype=torch.float64, device=dev) / NPHI


def _polar(images, T, r_max):
    """[n, L, L] -> bilinear polar samples [n, S, R, 256] at every integer shift."""
    n, L = images.shape[0], images.shape[-1]
    dev, pad = images.device, T + r_max + 3
    W = L + 2 * pad
    flat = torch.nn.functional.pad(images.double(), (pad,) * 4).reshape(n, -1)
    r = torch.arange(1, r_max + 1, dtype=torch.float64, device=dev)[:, None]
    x, y = r * torch.cos(_angles(dev)), r * torch.sin(_angles(dev))
    x0, y0 = torch.floor(x), torch.floor(y)
    fx, fy = x - x0, y - y0
    t = torch.arange(-T, T + 1, device=dev)
    shift = (t[:, None] * W + t[None, :]).reshape(-1, 1, 1)
    at = ((y0.long() + L // 2 + pad) * W + x0.long() + L // 2 + pad)[None] + shift
    idx = at.reshape(-1)
    out = 0.0
    for d, w in ((0, (1 - fx) * (1 - fy)), (1, fx * (1 - fy)), (W, (1 - fx) * fy), (W + 1, fx * fy)):
        out = out + flat[:, idx + d].reshape(n, *at.shape) * w
    return out


def _correlate(parts, refs, T, r_max):
    """CC table [n, K, M, S, 256] in 64 bits (both mirrors, references
    divided by their weighted ring norm)."""
    n, K = parts.shape[0], refs.shape[0]
    r = torch.arange(1, r_max + 1, dtype=torch.float64, device=parts.device)
    q = _polar(refs, 0, r_max)[:, 0]
    norm = torch.sqrt((r[None, :, None] * q * q).sum(dim=(1, 2)))
    Q = torch.fft.rfft(q / norm[:, None, None], dim=-1) * r[None, :, None]
    P = torch.fft.rfft(_polar(parts, T, r_max), dim=-1)
    S = P.shape[1]
    P = P.permute(3, 0, 1, 2).reshape(NPHI // 2 + 1, n * S, r_max).contiguous()
    Q = Q.permute(2, 1, 0).contiguous()
    out = torch.empty((n, K, 2, S, NPHI), dtype=torch.float64, device=parts.device)
    for m in (0, 1):
        G = torch.bmm(P.conj().resolve_conj().contiguous() if m == 0 else P, Q)
        G = G.reshape(NPHI // 2 + 1, n, S, K).permute(1, 3, 2, 0).contiguous()
        out[:, :, m] = torch.fft.irfft(G, n=NPHI, dim=-1)
    return out


def _align(parts, refs, T, r_max, cc2, psi_frac):
    """Best and runner-up CC, the winner's flat index and its sub-step angle."""
    N, K, S = parts.shape[0], refs.shape[0], (2 * T + 1) ** 2
    step = max(1, int(2.5e8 / (K * 2 * S * NPHI + S * r_max * NPHI * 4)))
    got = []
    for lo in range(0, N, step):
        cc = _correlate(parts[lo:lo + step], refs, T, r_max)
        n = cc.shape[0]
        flat = cc.reshape(n, -1)
        best, at = flat.max(dim=1)
        frac = second = None
        if psi_frac:
            a = at % NPHI
            row = cc.reshape(n, -1, NPHI)[torch.arange(n, device=cc.device), at // NPHI]
            v = [row.gather(1, ((a + d) % NPHI)[:, None])[:, 0] for d in (-1, 0, 1)]
            den = v[0] - 2 * v[1] + v[2]
            d = torch.where(den < 0, 0.5 * (v[0] - v[2]) / den, torch.zeros_like(den)).clamp(-0.5, 0.5)
            frac = ((NPHI - a) % NPHI - d) % NPHI
        if cc2:
            flat.scatter_(1, at[:, None], -math.inf)
            second = flat.max(dim=1).values
        got.append((best, at, second, frac))
    return [None if got[0][i] is None else torch.cat([g[i] for g in got]) for i in range(4)]


def _averages(parts, ref, sx, sy, psi, mirror, previous):
    """Mean of every class's particles, each warped back by its parameters."""
    L, K, dev = parts.shape[-1], previous.shape[0], parts.device
    sums = torch.zeros((K, L * L), dtype=torch.float64, device=dev)
    v = torch.arange(L, dtype=torch.float64, device=dev) - L // 2
    vx, vy = v[None, :].expand(L, L).reshape(-1), v[:, None].expand(L, L).reshape(-1)
    for lo in range(0, parts.shape[0], 2048):
        sl = slice(lo, lo + 2048)
        a = (2.0 * math.pi / NPHI) * psi[sl].double()[:, None]
        c, s = torch.cos(a), torch.sin(a)
        sign = (1 - 2 * mirror[sl].double())[:, None]
        X = L // 2 + sx[sl].double()[:, None] + c * vx - s * vy
        Y = L // 2 + sy[sl].double()[:, None] + sign * (s * vx + c * vy)
        # a border as wide as the furthest position (corner of the box plus shift)
        pad, W = L, 3 * L
        img = torch.nn.functional.pad(parts[sl].double(), (pad,) * 4).reshape(-1, W * W)
        x0, y0 = torch.floor(X), torch.floor(Y)
        fx, fy = X - x0, Y - y0
        at = (y0.long() + pad) * W + x0.long() + pad
        w = (img.gather(1, at) * (1 - fx) + img.gather(1, at + 1) * fx) * (1 - fy)
        w = w + (img.gather(1, at + W) * (1 - fx) + img.gather(1, at + W + 1) * fx) * fy
        sums.index_add_(0, ref[sl].long(), w)
    n = torch.bincount(ref.long(), minlength=K).to(torch.float64)[:, None]
    return torch.where(n > 0, sums / n.clamp(min=1), previous.double().reshape(K, -1)).reshape(K, L, L)


def exact(case, seed):
    data = _inputs(case, seed, torch.device("cuda", 0))
    refs, parts, truth = data[0]
    kind, T, r_max, dev = case["kind"], case["T"], case["r_max"], parts.device
    if kind == "averages":
        t = [torch.as_tensor(v, device=dev) for v in
             (truth.ref, truth.shift_x, truth.shift_y, truth.alpha * (NPHI / (2 * math.pi)), truth.mirror)]
        return dict(averages=_averages(parts, t[0], t[1], t[2], t[3].round().long() % NPHI, t[4], refs), counts=None)
    if kind in ("rfa", "classify"):
        S, none = (2 * T + 1) ** 2, torch.zeros(case["N"], dtype=torch.int64, device=dev)
        if kind == "rfa":
            avg = _averages(parts, none, none, none, none, none, parts[:1]).float()
        else:
            avg = refs
        before = None
        for i in range(case["iters"]):
            cc, at, second, _ = _align(parts, avg, T, r_max, kind == "rfa", False)
            a, s, m, k = at % NPHI, at // NPHI % S, at // (NPHI * S) % 2, at // (NPHI * S * 2)
            avg = _averages(parts, k, s % (2 * T + 1) - T, s // (2 * T + 1) - T, (NPHI - a) % NPHI, m, avg).float()
            now = at if kind == "rfa" else k
            if before is not None and bool((now == before).all()):
                break  # the loops stop at the first pass that changes nothing
            before = now
        return dict(cc=cc, cc2=second, average=avg[0]) if kind == "rfa" else dict(cc=cc, averages=avg)
    got = []
    for (refs, parts, _), (_, _, _, Ti, ri) in zip(data, _stacks(case)):
        cc, _, second, frac = _align(parts, refs, Ti, ri, case.get("cc2", False), case.get("psi_frac", False))
        got.append(dict({"cc": cc}, **({} if second is None else {"cc2": second}),
                        **({} if frac is None else {"psi_frac": frac})))
    return got if kind == "batch" else got[0]
