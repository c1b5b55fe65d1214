"""Performance cases of the library: what a user has it do for one layer.

Each case is a dict of plain values with a "kind" that names the step:

  refine   a whole refinement call from the host state (set-up and K sweeps);
  scales   layer set-up and one joint refit of the scales;
  codes    one code update (residual product, Gauss-Seidel decode) of a layer
           that is set up, with the scales refit to its codes;
  hessian  the calibration Hessian from chunks of tokens;
  gptq     the GPTQ-style host state;
  target   the propagation-corrected target: cross term and corrected weights;
  host     activation ordering, the round-to-nearest host on the reordered
           layer, and that state's row objectives;
  export   a refined layer to its deployed forms: canonical signs, weights in
           the model's dtype, packed codes.

Inputs are synthetic: heavy-tailed or Gaussian weights, input channels
correlated with their neighbours with a few outlier channels, a damped
Hessian.  Every random number comes from the seed.
"""

from __future__ import annotations

import math

import torch

from paper_2609_38599_amd import binding as jb

DAMP = 0.01        # relative diagonal damping of the Hessian
GROUPS_MAX = 128   # groups per row the library takes


def listed():
    return [
        # the smallest calls: launches and host latency count
        {"name": "refine_tiny", "kind": "refine", "rows": 64, "cols": 256, "g": 64, "bits": 3,
         "sweeps": 5, "tau": -1.0, "host": "rtn"},
        # the benchmark's layer, a fixed budget of sweeps
        {"name": "refine_attn", "kind": "refine", "rows": 4096, "cols": 4096, "g": 128, "bits": 3,
         "sweeps": 10, "tau": -1.0, "host": "rtn"},
        # a wide MLP layer from a GPTQ-style host with the stopping rule on
        {"name": "refine_mlp_stop", "kind": "refine", "rows": 14336, "cols": 4096, "g": 64,
         "bits": 3, "sweeps": 20, "tau": 1e-5, "host": "gptq"},
        # a down projection: many groups a row, a Hessian of 11008 channels
        {"name": "scales_down", "kind": "scales", "rows": 4096, "cols": 11008, "g": 128, "bits": 3},
        # a small ragged layer, short groups, wide codes
        {"name": "scales_ragged", "kind": "scales", "rows": 611, "cols": 1312, "g": 32, "bits": 8},
        # an up projection at 4 bits
        {"name": "codes_up", "kind": "codes", "rows": 11008, "cols": 4096, "g": 128, "bits": 4},
        # calibration inputs kept in fp32, and in the models' bf16 (a larger
        # set), a few sequences a chunk
        {"name": "hessian_f32", "kind": "hessian", "cols": 4096, "tokens": 16384, "chunk": 8192,
         "dtype": "float32"},
        {"name": "hessian_bf16", "kind": "hessian", "cols": 4096, "tokens": 65536, "chunk": 8192,
         "dtype": "bfloat16"},
        # the GPTQ-style host of an attention projection
        {"name": "gptq_attn", "kind": "gptq", "rows": 4096, "cols": 4096, "g": 128, "bits": 3},
        # one calibration sequence's cross term and the corrected weights
        {"name": "target_attn", "kind": "target", "rows": 4096, "cols": 4096, "g": 128, "bits": 3,
         "tokens": 2048, "mu": 0.5},
        # the round-to-nearest start of a mid-sized layer, reordered
        {"name": "host_mid", "kind": "host", "rows": 1000, "cols": 2752, "g": 32, "bits": 4},
        # write-back of a reordered layer in the models' dtype
        {"name": "export_up", "kind": "export", "rows": 11008, "cols": 4096, "g": 128, "bits": 4,
         "dtype": "bfloat16", "perm": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["refine", "refine", "scales", "codes", "hessian", "hessian", "gptq",
                       "target", "host", "export"])
    if kind == "hessian":
        dtype = rng.choice(["float32", "bfloat16"])
        cols = 8 * _log(rng, 16, 1376)
        # at most the work of the largest listed Hessian of that dtype
        most = 4096 * 4096 * (16384 if dtype == "float32" else 65536) // (cols * cols)
        tokens = _log(rng, 128, max(256, min(65536, most)))
        chunk = min(tokens, _log(rng, 128, 16384))
        chunk = max(chunk, -(-tokens // 64))
        return {"kind": kind, "cols": cols, "tokens": tokens, "chunk": chunk, "dtype": dtype}
    g = rng.choice([32, 64, 128, 128])
    wide = 11008 if kind in ("scales", "codes", "host", "export") else 4096
    cols = g * _log(rng, max(2, 256 // g), min(GROUPS_MAX, wide // g))
    most = 4096 if kind in ("gptq", "target") else 14336
    most = min(most, 4096 * 4096 * 11008 // (cols * cols))
    rows = _log(rng, 16, max(32, most))
    case = {"kind": kind, "rows": rows, "cols": cols, "g": g, "bits": rng.choice([2, 3, 3, 4, 4, 8])}
    if kind == "refine":
        case["sweeps"] = rng.randint(3, 20)
        case["tau"] = rng.choice([-1.0, 1e-5])
        case["host"] = rng.choice(["rtn", "gptq"])
    elif kind == "target":
        case["tokens"] = _log(rng, 256, 2048)
        case["mu"] = rng.choice([0.0, 0.25, 0.5])
    elif kind == "export":
        case["dtype"] = rng.choice(["float32", "float16", "bfloat16"])
        case["perm"] = rng.choice([True, False])
    return case


# ---- inputs ----

def _gen(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    return gen


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32)


def _weights(gen, rows, cols):
    """Student-t with 5 degrees of freedom, standard deviation 0.02."""
    w = _randn(gen, rows, cols)
    chi = torch.zeros_like(w)
    for _ in range(5):
        chi += _randn(gen, rows, cols).square_()
    return (w / (chi / 5.0).sqrt_() * (0.02 * math.sqrt(3.0 / 5.0))).contiguous()


def _channel_scale(gen, cols):
    """One channel in a hundred is an outlier, twenty times the others."""
    u = torch.rand(cols, generator=gen, device="cuda")
    return torch.where(u < 0.01, 20.0, 1.0)


def _tokens(gen, m, cols, scale):
    """m tokens: channels correlated with their neighbours (0.6 a step, cut
    off after twelve), outlier channels scaled."""
    rho, taps = 0.6, 12
    z = _randn(gen, m, cols + taps)
    x = z[:, taps:].clone()
    for k in range(1, taps):
        x.add_(z[:, taps - k:taps - k + cols], alpha=rho ** k)
    return x.mul_(scale * math.sqrt(1.0 - rho * rho)).contiguous()


def _hessian_input(gen, cols):
    """A damped fp32 Hessian (exactly symmetric) of 2 cols tokens."""
    scale = _channel_scale(gen, cols)
    m = 2 * cols
    X = _tokens(gen, m, cols, scale)
    H = X.t() @ X
    H.div_(float(m))
    H = 0.5 * (H + H.t())
    H.diagonal().add_(DAMP * H.diagonal().mean())
    return H.contiguous(), scale


def _params(case, sweeps=1, tau=-1.0):
    return jb.make_params(case["rows"], case["cols"], case["g"], case["bits"], sweeps=sweeps,
                          tau=tau)


def _scratch(nbytes):
    raw = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
    off = (-raw.data_ptr()) % 256
    return raw[off:off + nbytes]


def prepare(case, seed):
    gen = _gen(seed)
    kind = case["kind"]
    st = {"case": case}
    if kind == "hessian":
        dtype = getattr(torch, case["dtype"])
        scale = _channel_scale(gen, case["cols"])
        left, chunks = case["tokens"], []
        while left > 0:
            m = min(left, case["chunk"])
            chunks.append(_tokens(gen, m, case["cols"], scale).to(dtype))
            left -= m
        st["chunks"] = chunks
        return st
    rows, cols, g = case["rows"], case["cols"], case["g"]
    p = _params(case, case.get("sweeps", 1), case.get("tau", -1.0))
    st["p"] = p
    st["W"] = _weights(gen, rows, cols)
    if kind == "export":
        # a refined layer: codes, scales (a few of them negative), zero points
        # and the order its columns are in
        G, top = cols // g, 1 << case["bits"]
        z = _randn(gen, rows, cols).mul_(top / 5.0).add_(top / 2.0)
        st["codes"] = z.round_().clamp_(0, top - 1).to(torch.uint8)
        s = torch.rand(rows, G, generator=gen, device="cuda") * 0.01 + 0.005
        neg = torch.rand(rows, G, generator=gen, device="cuda") < 0.02
        st["scales"] = torch.where(neg, -s, s).contiguous()
        st["zeros"] = torch.randint(0, top, (rows, G), generator=gen, device="cuda",
                                    dtype=torch.int32)
        st["perm"] = (torch.randperm(cols, generator=gen, device="cuda").to(torch.int32)
                      if case["perm"] else None)
        del st["W"]
        return st
    st["H"], scale = _hessian_input(gen, cols)
    if kind == "target":
        m = case["tokens"]
        st["X"] = _tokens(gen, m, cols, scale)
        # what the layer receives once the layers before it are quantized
        st["Xq"] = (st["X"] * (1.0 + 0.1 * _randn(gen, m, cols))
                    + 0.02 * scale * _randn(gen, m, cols)).contiguous()
        st["ws"] = _scratch(int(jb.load_library().jarq_qep_workspace_bytes(p)))
        return st
    if kind == "gptq":
        st["ws"] = _scratch(int(jb.load_library().jarq_gptq_workspace_bytes(p)))
        return st
    # a workspace with defined contents (a program allocates it once and
    # keeps it for many calls)
    st["ws"] = jb.alloc_workspace(p).zero_()
    if kind == "host":
        return st
    if case.get("host", "rtn") == "gptq":
        st["codes"], st["scales"], st["zeros"] = jb.gptq(p, st["W"], st["H"])
    else:
        st["codes"], st["scales"], st["zeros"] = jb.rtn(p, st["W"])
    if kind == "codes":
        jb.prepare(p, st["W"], st["H"], st["ws"])
        jb.scale_step(p, st["H"], st["codes"], st["scales"], st["zeros"], st["ws"])
    return st


# ---- one pass ----

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "hessian":
        # the mean over the tokens, damped
        return jb.hessian(st["chunks"], case["cols"], alpha=1.0 / case["tokens"], damp=DAMP)
    p = st["p"]
    if kind == "refine":
        codes, scales = st["codes"].clone(), st["scales"].clone()
        jb.refine(p, st["W"], st["H"], codes, scales, st["zeros"], st["ws"], want_stats=False)
        return {"codes": codes, "scales": scales}
    if kind == "scales":
        scales = st["scales"].clone()
        jb.prepare(p, st["W"], st["H"], st["ws"])
        jb.scale_step(p, st["H"], st["codes"], scales, st["zeros"], st["ws"])
        return {"scales": scales}
    if kind == "codes":
        codes = st["codes"].clone()
        jb.code_step(p, st["W"], st["H"], codes, st["scales"], st["zeros"], st["ws"])
        return {"codes": codes}
    if kind == "gptq":
        codes, scales, zeros = jb.gptq(p, st["W"], st["H"], ws=st["ws"])
        return {"codes": codes, "scales": scales, "zeros": zeros}
    if kind == "target":
        d = case["cols"]
        D = torch.zeros(d, d, dtype=torch.float64, device="cuda")
        jb.cross_accumulate(st["Xq"], st["X"], D, alpha=1.0 / case["tokens"])
        W = jb.qep_correct(p, st["W"], st["H"], D, case["mu"], ws=st["ws"])
        return {"D": D, "W": W}
    if kind == "host":
        perm = jb.act_order(st["H"])
        Wp, Hp = jb.permute(p, perm, st["W"], st["H"])
        codes, scales, zeros = jb.rtn(p, Wp)
        obj = jb.objective(p, Wp, Hp, codes, scales, zeros, st["ws"])
        return {"perm": perm, "Wp": Wp, "Hp": Hp, "codes": codes, "scales": scales,
                "zeros": zeros, "objective": obj}
    if kind == "export":
        codes, scales, zeros = st["codes"].clone(), st["scales"].clone(), st["zeros"].clone()
        jb.canonicalize(p, codes, scales, zeros)
        w = jb.dequantize(p, codes, scales, zeros, dtype=getattr(torch, case["dtype"]),
                          perm=st["perm"])
        packed = jb.pack_codes(p, codes)
        return {"scales": scales, "zeros": zeros, "w": w, "packed": packed}
    raise ValueError(kind)


# ---- what a pass cannot do without ----

def work(case):
    kind = case["kind"]
    d = case["cols"]
    if kind == "hessian":
        m = case["tokens"]
        size = 4 if case["dtype"] == "float32" else 2
        return {"bytes": m * d * size + 4 * d * d, "flops": m * d * (d + 1)}
    R, g, b = case["rows"], case["g"], case["bits"]
    G = d // g
    n = R * d
    layer = 4 * n + 4 * d * d             # W and H
    state = n + 8 * R * G                 # codes, scales, zero points
    factor = d * d * g // 3 + d * d * g   # factors of the diagonal blocks, M = L^-1 H
    gram = n * (d + g) + n * G            # half the Gram entries, and their products with c
    solve = R * G * G * G // 3
    resid = 2 * n * d                     # the residual product
    decode = 2 * n * g                    # objective and back substitution
    if kind == "refine":
        return {"bytes": layer + 2 * state,
                "flops": factor + 2 * n * d + case["sweeps"] * (gram + solve + resid + decode)}
    if kind == "scales":
        return {"bytes": layer + state + 4 * R * G, "flops": factor + 2 * n * d + gram + solve}
    if kind == "codes":
        return {"bytes": layer + state + n, "flops": resid + decode}
    if kind == "gptq":
        return {"bytes": layer + state, "flops": d * d * d // 3 + n * d + 2 * n * g}
    if kind == "target":
        m = case["tokens"]
        return {"bytes": layer + 8 * m * d + 8 * d * d + 4 * n,
                "flops": 2 * m * d * d + d * d * d // 3 + 4 * n * d}
    if kind == "host":
        return {"bytes": 2 * layer + state + 8 * R, "flops": 2 * n * d}
    if kind == "export":
        size = 4 if case["dtype"] == "float32" else 2
        return {"bytes": state + size * n + 4 * R * ((d * b + 31) // 32) + 8 * R * G,
                "flops": 2 * n}
    raise ValueError(kind)


def tolerance(case):
    kind = case["kind"]
    if kind == "hessian":
        # fp32 sums of at most 256 tokens, added in fp64, rounded to fp32:
        # up to 1.2e-7 from the 64-bit build
        return {"rel": 5e-7, "max": 1e-5}
    if kind == "refine":
        # A decision within rounding of its boundary may go either way and
        # takes its row along another, equally good descent: the same layer
        # with every rounding changed (W and the scales times 1.1) differs in
        # up to 1.25e-2 of the codes and 7e-3 in the scales.
        return {"rel": 3e-2, "differ": 5e-2}
    if kind == "scales":
        # 1.5e-6 between such a pair, 1.1e-6 from the 64-bit solve
        return {"rel": 6e-6, "max": 1e-4}
    if kind == "codes":
        # 2.5e-3 between such a pair (8-bit codes)
        return {"rel": 0.0, "differ": 1e-2}
    if kind == "gptq":
        # fp64 throughout: a code changes only at a tie, and then its row
        return {"rel": 1e-5, "differ": 1e-5}
    if kind == "target":
        # the cross term 2.6e-7 from its 64-bit build, the weights 1.7e-7
        return {"rel": 1e-6, "max": 1e-4}
    if kind == "host":
        # the objective of fp32 products, 2.9e-7 from its 64-bit value
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.0}
    return "exact"


# ---- the same in 64 bits ----

def exact(case, seed):
    """run()'s outputs in float64 with plain torch; None for the codes (whole
    numbers, which depend on ties) and for a refinement, whose trajectory
    forks at decisions within rounding of their boundary."""
    kind = case["kind"]
    if kind in ("refine", "codes"):
        return None
    st = prepare(case, seed)
    d = case["cols"]
    if kind == "hessian":
        H = torch.zeros(d, d, dtype=torch.float64, device="cuda")
        for X in st["chunks"]:
            X = X.double()
            H += X.t() @ X
        H /= case["tokens"]
        H.diagonal().add_(DAMP * H.diagonal().mean())
        return H
    R, g, top = case["rows"], case["g"], float((1 << case["bits"]) - 1)
    G = d // g
    if kind == "export":
        s, z, q = st["scales"], st["zeros"], st["codes"]
        neg = s < 0
        w = (q.view(R, G, g).double() - z.double()[:, :, None]) * s.double()[:, :, None]
        w = w.view(R, d)
        if st["perm"] is not None:
            out = torch.empty_like(w)
            out[:, st["perm"].long()] = w
            w = out
        return {"scales": s.double().abs(), "zeros": None, "w": w, "packed": None}
    W, H = st["W"].double(), st["H"].double()
    if kind == "scales":
        C = (st["codes"].view(R, G, g).double() - st["zeros"].double()[:, :, None])
        flat = C.reshape(R, d)
        A = torch.empty(R, G, G, dtype=torch.float64, device="cuda")
        rhs = ((W @ H).view(R, G, g) * C).sum(2)
        for a in range(G):
            T = flat[:, a * g:(a + 1) * g] @ H[a * g:(a + 1) * g, :]
            A[:, a, :] = (T.view(R, G, g) * C).sum(2)
        s = torch.linalg.solve(A.cpu(), rhs.cpu()[:, :, None])[:, :, 0]
        return {"scales": s}
    if kind == "target":
        Xq, X = st["Xq"].double(), st["X"].double()
        D = Xq.t() @ (X - Xq) / case["tokens"]
        T = W @ D.t().contiguous()
        L = torch.linalg.cholesky(H.cpu())
        Z = torch.cholesky_solve(T.t().contiguous().cpu(), L).t().contiguous().cuda()
        return {"D": D, "W": W + (1.0 - case["mu"]) * Z}
    if kind == "host":
        perm = torch.sort(H.diagonal(), descending=True, stable=True).indices
        Wp = W[:, perm]
        Hp = H[perm][:, perm]
        lo = Wp.view(R, G, g).amin(2).clamp(max=0.0)
        hi = Wp.view(R, G, g).amax(2).clamp(min=0.0)
        s = torch.where(hi > lo, (hi - lo) / top, torch.ones_like(hi))
        s32 = s.float().double()
        z = torch.round(-lo / s32).clamp(0.0, top)
        q = (torch.round(Wp.view(R, G, g) / s32[:, :, None]) + z[:, :, None]).clamp(0.0, top)
        E = Wp - (s32[:, :, None] * (q - z[:, :, None])).view(R, d)
        return {"perm": None, "Wp": Wp, "Hp": Hp, "codes": None, "scales": s, "zeros": None,
                "objective": ((E @ Hp) * E).sum(1)}
    if kind == "gptq":
        # the usual recursion on the upper factor of the inverse
        Hinv = torch.cholesky_inverse(torch.linalg.cholesky(H.cpu()))
        U = torch.linalg.cholesky(Hinv, upper=True).cuda()
        scales = torch.empty(R, G, dtype=torch.float64, device="cuda")
        for i in range(G):
            c0, c1 = i * g, (i + 1) * g
            blk = W[:, c0:c1]
            lo, hi = blk.amin(1).clamp(max=0.0), blk.amax(1).clamp(min=0.0)
            s = torch.where(hi > lo, (hi - lo) / top, torch.ones_like(hi))
            scales[:, i] = s
            s32 = s.float().double()
            z = torch.round(-lo / s32).clamp(0.0, top)
            err = torch.empty(R, g, dtype=torch.float64, device="cuda")
            blk = blk.clone()
            for k in range(g):
                w = blk[:, k]
                q = (torch.round(w / s32) + z).clamp(0.0, top)
                e = (w - s32 * (q - z)) / U[c0 + k, c0 + k]
                err[:, k] = e
                if k + 1 < g:
                    blk[:, k + 1:] -= e[:, None] * U[c0 + k, c0 + k + 1:c1][None, :]
            if c1 < d:
                W[:, c1:] -= err @ U[c0:c1, c1:]
        return {"codes": None, "scales": scales, "zeros": None}
    raise ValueError(kind)
