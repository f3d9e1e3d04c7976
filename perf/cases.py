"""The work a user of sga has it do, as measurable cases over the public entry points.

A case names an operation, a mask family with its parameters, and the shape of the tensors:

  step       build_mask, then attention_forward on the CSR: a program that meets a new mask
  prepared   attention_forward_prepared: one fixed mask, many layers and steps
  implicit   attention_forward_implicit: neighbours from index arithmetic, no stored graph
  compose    implicit local, implicit non-local and (bigbird) a prepared CSR call on one
             (O, lse) state: the sequence of Section V-F of the paper
  static     attention_forward_static: a small call that allocates nothing

Tensors are [H][L][d]; fp32 inputs are N(0, 1), fp16 inputs N(0, 1) / 2, the verification
protocol's are U[0, 1) (Section V-A).  Every output buffer and workspace is the caller's and is
kept from pass to pass, as a model's would be.
"""
import math

import torch

import paper_2502_01659_amd as sga
from sga_inputs import (MaskSpec, KIND_SLIDING, KIND_DILATED, KIND_GLOBAL_LOCAL, KIND_BIGBIRD,
                        KIND_NONLOCAL, KIND_DILATED_2D)

_DTYPE = {"f32": torch.float32, "f16": torch.float16}
_GOLD = 0x9E3779B97F4A7C15
_U64 = (1 << 64) - 1


def _case(name, op, mask, dtype, H, L, d, **params):
    return {"name": name, "op": op, "mask": mask, "dtype": dtype, "H": H, "L": L, "d": d, **params}


def listed():
    return [
        # the smallest call: the paper's verification protocol (Section V-A), a Bernoulli mask
        _case("verify_256_d32_f32", "static", "random", "f32", 1, 256, 32, density=0.1),
        # a short sequence whose mask is new: launches and latency count, not rates
        _case("sliding_4k_f32", "step", "sliding", "f32", 1, 4096, 64, window=32),
        # a Longformer layer in steady state: window, global rows and columns, 8 heads
        _case("longformer_64k_f32", "prepared", "global_local", "f32", 8, 65536, 64, window=128, n_global=16),
        # a BigBird-style mask of a million tokens, built and used once
        _case("bigbird_1m_f16", "step", "bigbird", "f16", 4, 1 << 20, 64, block=64, window_blocks=1,
              n_global_blocks=2, n_random_blocks=3),
        # a dilated window of a million tokens without an index
        _case("dilated_1m_f16", "implicit", "dilated", "f16", 4, 1 << 20, 64, window=64, stride=2),
        # extreme length, narrow window: the memory system's case
        _case("sliding_32m_f16", "implicit", "sliding", "f16", 1, 32_000_000, 64, window=16),
        # the shortest of the long-context runs (Table III): a wide band at d = 64
        _case("band_1p6m_f16", "implicit", "sliding", "f16", 1, 1_600_000, 64, window=1359),
        # a current model's sliding-window layer: 32 heads of 128 channels
        _case("band_32k_d128_f16", "implicit", "sliding", "f16", 32, 32768, 128, window=2048),
        # the microbenchmark's dense end (Section V-C) at d = 256, a ragged length
        _case("band_16k_d256_f32", "implicit", "sliding", "f32", 1, 16301, 256, window=815),
        # the microbenchmark's uniformly random CSR: irregular neighbours
        _case("random_24k_f32", "prepared", "random", "f32", 1, 24576, 64, density=0.1),
        # a Longformer layer as two calls on one state, 16-bit storage
        _case("longformer_calls_64k_f16", "compose", "global_local", "f16", 8, 65536, 64, window=128, n_global=16),
        # the BigBird model mask of Section V-F as three calls on one state, a ragged length
        _case("bigbird_calls_35k_f32", "compose", "bigbird_model", "f32", 1, 35000, 64, window=50, n_global=3,
              density=0.001),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        case = _draw_any(rng)
        w = work(case)
        if w["bytes"] <= 1.7e10 and w["flops"] <= (2.0e12 if case["dtype"] == "f16" else 1.0e11):
            return case


def _draw_any(rng):
    family = rng.choice(("verify", "window_csr", "longformer", "bigbird", "window", "band", "random", "calls"))
    dtype = rng.choice(("f32", "f16"))
    c = {"dtype": dtype, "H": rng.choice((1, 1, 2, 4, 8)), "d": 64}
    if family == "verify":
        c.update(op="static", mask="random", L=_log(rng, 100, 3000), H=1, d=rng.choice((32, 64)),
                 density=rng.choice((0.01, 0.1, 0.5)))
    elif family == "window_csr":
        c.update(op=rng.choice(("step", "prepared")), mask="sliding", L=_log(rng, 2000, 400_000),
                 window=_log(rng, 8, 400), d=rng.choice((64, 64, 128)))
    elif family == "longformer":
        c.update(op=rng.choice(("step", "prepared")), mask="global_local", L=_log(rng, 4000, 300_000),
                 window=_log(rng, 32, 300), n_global=rng.randint(1, 32), d=rng.choice((64, 64, 128)))
    elif family == "bigbird":
        block = rng.choice((32, 64, 64))
        c.update(op=rng.choice(("step", "prepared")), mask="bigbird", L=block * _log(rng, 64, 16384), block=block,
                 window_blocks=1, n_global_blocks=rng.randint(1, 3), n_random_blocks=rng.randint(1, 4),
                 d=rng.choice((64, 64, 128)))
    elif family == "window":
        stride = rng.choice((1, 1, 2, 3))
        c.update(op="implicit", mask="dilated" if stride > 1 else "sliding", L=_log(rng, 10_000, 20_000_000),
                 window=_log(rng, 8, 130), d=rng.choice((64, 64, 128)))
        if stride > 1:
            c["stride"] = stride
    elif family == "band":
        d = rng.choice((64, 128, 256))
        c.update(op="implicit", L=_log(rng, 4000, 1_600_000), d=d)
        if rng.random() < 0.25:
            c.update(mask="dilated_2d", block=_log(rng, 100, 4000), stride=2)
        else:
            c.update(mask="sliding", window=_log(rng, 200, 2100))
        if c["L"] < 50_000:
            c["H"] = rng.choice((1, 4, 16, 32))
    elif family == "random":
        c.update(op="prepared", mask="random", L=_log(rng, 3000, 24576), H=1, d=rng.choice((64, 64, 128)),
                 density=rng.choice((0.01, 0.1, 0.25, 0.5)))
    else:
        c.update(op="compose", mask=rng.choice(("global_local", "bigbird_model")), L=_log(rng, 8000, 50_000),
                 window=_log(rng, 32, 150), n_global=rng.randint(1, 16))
        if c["mask"] == "bigbird_model":
            c.update(H=1, density=0.001)
        else:
            c["L"] *= rng.choice((1, 4))
    return c


# ---- masks ------------------------------------------------------------------------------------------
def _scale(case):
    return 1.0 / math.sqrt(case["d"])


def _spec(case, seed):
    L = case["L"]
    kind = case["mask"]
    if kind == "sliding":
        return MaskSpec(KIND_SLIDING, L, window=case["window"])
    if kind == "dilated":
        return MaskSpec(KIND_DILATED, L, window=case["window"], stride=case["stride"])
    if kind == "dilated_2d":
        return MaskSpec(KIND_DILATED_2D, L, block=case["block"], stride=case["stride"])
    if kind == "global_local":
        return MaskSpec(KIND_GLOBAL_LOCAL, L, window=case["window"], n_global=case["n_global"])
    if kind == "bigbird":
        return MaskSpec(KIND_BIGBIRD, L, block=case["block"], window_blocks=case["window_blocks"],
                        n_global_blocks=case["n_global_blocks"], n_random_blocks=case["n_random_blocks"],
                        seed=seed + 3)
    raise ValueError(kind)


def _random_rows(case, seed):
    """Row blocks (first row, bool [rows, L]) of the uniformly random part of a mask.  In a model's
    BigBird mask the edges of the local and global parts are left out: those have calls of their own."""
    L = case["L"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 7)
    for r0 in range(0, L, 1024):
        rows = torch.rand((min(1024, L - r0), L), generator=g, device="cuda") < case["density"]
        if case["mask"] == "bigbird_model":
            rows &= ~_longformer_rows(case, r0, rows.shape[0])
        yield r0, rows


def _longformer_rows(case, r0, n):
    i = torch.arange(r0, r0 + n, device="cuda")[:, None]
    j = torch.arange(case["L"], device="cuda")[None, :]
    return ((i - j).abs() <= case["window"]) | (i < case["n_global"]) | (j < case["n_global"])


def _random_csr(case, seed):
    row_ptr = torch.zeros(case["L"] + 1, dtype=torch.int64, device="cuda")
    counts, cols = [], []
    for _, rows in _random_rows(case, seed):
        counts.append(rows.sum(dim=1))
        cols.append(rows.nonzero()[:, 1].to(torch.int32))
    row_ptr[1:] = torch.cat(counts).cumsum(0)
    return row_ptr, torch.cat(cols).contiguous()


def _edges(case):
    """Edges of the mask (of the expected mask, where it is random) per head."""
    L, kind = case["L"], case["mask"]

    def band(n, w):     # pairs |i - j| <= w of a class of n tokens
        w = min(w, n - 1)
        return n * (2 * w + 1) - w * (w + 1)
    if kind == "sliding":
        return band(L, case["window"])
    if kind == "dilated":
        s = case["stride"]
        return sum(band((L - r + s - 1) // s, case["window"]) for r in range(s))
    if kind == "dilated_2d":
        b, s = case["block"], case["stride"]
        return (L // b) * ((b + s - 1) // s) ** 2 + ((L % b + s - 1) // s) ** 2
    if kind in ("global_local", "bigbird_model"):
        g, w = min(case["n_global"], L), case["window"]
        inside = L * L - (L - g) * (L - g) + band(max(L - g, 1), w)
        return inside + (int(case["density"] * (L * L - inside)) if kind == "bigbird_model" else 0)
    if kind == "bigbird":
        nb = L // case["block"]
        G, W = case["n_global_blocks"], case["window_blocks"]
        n = G * nb
        for b in range(G, nb):
            own = set(range(max(0, b - W), min(nb, b + W + 1))) | set(range(G)) if b < G + W + 1 or b + W >= nb else None
            n += (len(own) if own is not None else 2 * W + 1 + G) + case["n_random_blocks"]
        return n * case["block"] ** 2
    return int(case["density"] * L * L)


# ---- prepare, run -------------------------------------------------------------------------------------
def _qkv(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt, shape = _DTYPE[case["dtype"]], (case["H"], case["L"], case["d"])
    out = []
    for _ in range(3):
        if case["op"] == "static":
            x = torch.rand(shape, generator=g, device="cuda").to(dt)
        else:
            x = torch.randn(shape, generator=g, device="cuda", dtype=dt)
            if case["dtype"] == "f16":
                x.mul_(0.5)
        out.append(x)
    return out


def prepare(case, seed):
    H, L, d, dtype = case["H"], case["L"], case["d"], case["dtype"]
    Q, K, V = _qkv(case, seed)
    s = {"op": case["op"], "Q": Q, "K": K, "V": V, "O": torch.empty_like(Q), "scale": _scale(case)}
    if case["op"] == "step":
        s["spec"] = _spec(case, seed)
        s["ws"] = sga.alloc_workspace(L, H, d, dtype, sga.mask_nnz(s["spec"]))
    elif case["op"] == "prepared":
        s["rp"], s["ci"] = _random_csr(case, seed) if case["mask"] == "random" else sga.build_mask(_spec(case, seed))
        s["ws"] = sga.alloc_workspace(L, H, d, dtype, s["ci"].numel())
        s["plan"] = sga.graph_prepare(s["rp"], s["ci"], H, d, dtype, s["ws"])
    elif case["op"] == "implicit":
        s["spec"] = _spec(case, seed)
        s["ws"] = sga.alloc_workspace(L, H, d, dtype, -1)
    elif case["op"] == "compose":
        s["lse"] = torch.empty((H, L), dtype=torch.float32, device="cuda")
        s["local"] = MaskSpec(KIND_SLIDING, L, window=case["window"])
        s["nonlocal"] = MaskSpec(KIND_NONLOCAL, L, window=case["window"], n_global=case["n_global"])
        s["ws"] = sga.alloc_workspace(L, H, d, dtype, -1)
        if case["mask"] == "bigbird_model":
            s["rp"], s["ci"] = _random_csr(case, seed)
            s["csr_ws"] = sga.alloc_workspace(L, H, d, dtype, s["ci"].numel())
            s["plan"] = sga.graph_prepare(s["rp"], s["ci"], H, d, dtype, s["csr_ws"])
    else:
        s["rp"], s["ci"] = _random_csr(case, seed)
        s["lse"] = torch.empty((H, L), dtype=torch.float32, device="cuda")
        s["code"] = 0 if dtype == "f32" else 1
        sga.sga_static_scratch_init()
    return s


def run(s):
    op, Q, K, V, O, scale = s["op"], s["Q"], s["K"], s["V"], s["O"], s["scale"]
    if op == "step":
        rp, ci = sga.build_mask(s["spec"])
        return {"O": sga.attention_forward(Q, K, V, rp, ci, scale, O=O, workspace=s["ws"]), "row_ptr": rp, "col_idx": ci}
    if op == "prepared":
        return {"O": sga.attention_forward_prepared(Q, K, V, s["rp"], s["ci"], scale, s["plan"], s["ws"], O=O)}
    if op == "implicit":
        return {"O": sga.attention_forward_implicit(Q, K, V, s["spec"], scale, O=O, workspace=s["ws"])}
    if op == "compose":
        lse = s["lse"]
        sga.attention_forward_implicit(Q, K, V, s["local"], scale, O=O, lse=lse, workspace=s["ws"])
        sga.attention_accumulate_implicit(Q, K, V, s["nonlocal"], scale, O, lse, workspace=s["ws"])
        if "plan" in s:
            sga.attention_accumulate_prepared(Q, K, V, s["rp"], s["ci"], scale, s["plan"], s["csr_ws"], O, lse)
        return {"O": O, "lse": lse}
    H, L, d = Q.shape
    st = sga.sga_attention_forward_static(
        Q.data_ptr(), K.data_ptr(), V.data_ptr(), s["rp"].data_ptr(), s["ci"].data_ptr(), O.data_ptr(), L, H, d,
        scale, torch.cuda.current_stream().cuda_stream, s["code"], s["lse"].data_ptr(), s["ci"].numel(), sga.PATH_AUTO)
    if st != 0:
        raise sga.SgaError(st, "sga_attention_forward_static")
    return {"O": O, "lse": s["lse"]}


def work(case):
    """Each input read once and each output written once (Q, K, V, O, the index arrays an
    operation is given or has to return), 2d multiply-adds per edge and head."""
    H, L, d, E = case["H"], case["L"], case["d"], _edges(case)
    b = 4 * H * L * d * (4 if case["dtype"] == "f32" else 2)
    if case["op"] in ("step", "static") or case["mask"] == "random":
        b += 4 * E + 8 * (L + 1)
    elif case["op"] == "prepared":
        b += 8 * (L + 1)
    elif case["mask"] == "bigbird_model":
        b += int(4 * case["density"] * L * L) + 8 * (L + 1)
    if case["op"] in ("compose", "static"):
        b += 4 * H * L
    return {"bytes": b, "flops": 4 * d * H * E}


def tolerance(case):
    """About four times the largest error against `exact` that was seen over the ranges of `draw`.
    fp32: sums of up to 65,536 terms and exp2 to a unit in the last place.  fp16: the numerators of
    the softmax and O are rounded to 11 bits, in a composed state O once per call."""
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-4, "differ": 0.0}
    return {"rel": 1.6e-3, "max": 2e-2, "differ": 0.0}


# ---- the definition in 64 bits ------------------------------------------------------------------------
def _softmax_v(Q, K, V, ok, scale):
    """Q [..., n, d], K and V [..., m, d], ok [..., n, m] -> (O, lse); rows without a neighbour: 0 and -inf."""
    S = torch.matmul(Q, K.transpose(-1, -2).contiguous()).mul_(scale)
    S.masked_fill_(~ok, -math.inf)
    lse = torch.logsumexp(S, dim=-1)
    P = S.sub_(torch.where(lse == -math.inf, torch.zeros_like(lse), lse)[..., None]).exp_()
    return torch.matmul(P, V), lse


def _band(Q, K, V, w, scale, extra=0):
    """|i - j| <= w over one class [H, n, d]; with extra = g also the first g keys (for rows >= g)."""
    H, n, d = Q.shape
    B = min(n, 128 if w < 200 else 1024)
    m = min(B + 2 * w, n + B)
    O, lse = torch.empty_like(Q, dtype=torch.float64), torch.empty((H, n), dtype=torch.float64, device=Q.device)
    nb = (n + B - 1) // B
    step = max(1, int(1.5e8 / (H * B * (m + extra))), )
    for b0 in range(0, nb, step):
        b1 = min(nb, b0 + step)
        i = torch.arange(b0, b1, device=Q.device)[:, None] * B + torch.arange(B, device=Q.device)[None, :]
        first = (torch.arange(b0, b1, device=Q.device) * B - w).clamp(min=0)
        j = first[:, None] + torch.arange(m, device=Q.device)[None, :]
        ok = ((i[:, :, None] - j[:, None, :]).abs() <= w) & (j[:, None, :] < n)
        jc, ic = j.clamp(max=n - 1), i.clamp(max=n - 1)
        Kg, Vg = K[:, jc].double(), V[:, jc].double()
        if extra:
            ok &= j[:, None, :] >= extra
            ok = torch.cat((torch.ones((b1 - b0, B, extra), dtype=torch.bool, device=Q.device), ok), dim=2)
            Kg = torch.cat((K[:, None, :extra].double().expand(H, b1 - b0, extra, d), Kg), dim=2)
            Vg = torch.cat((V[:, None, :extra].double().expand(H, b1 - b0, extra, d), Vg), dim=2)
        o, l = _softmax_v(Q[:, ic].double(), Kg, Vg, ok[None], scale)
        lo, hi = b0 * B, min(n, b1 * B)
        O[:, lo:hi] = o.reshape(H, -1, d)[:, :hi - lo]
        lse[:, lo:hi] = l.reshape(H, -1)[:, :hi - lo]
    return O, lse


def _dense_rows(Q, K, V, ok, r0, O, lse, scale):
    n = ok.shape[0]
    Qd, Kd, Vd = Q[:, r0:r0 + n].double(), K.double(), V.double()
    O[:, r0:r0 + n], lse[:, r0:r0 + n] = _softmax_v(Qd, Kd, Vd, ok[None], scale)


def _mix64(z):
    z &= _U64
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _U64
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _U64
    return z ^ (z >> 31)


def _bigbird_blocks(case, seed):
    """Key blocks of every query block >= n_global_blocks, padded with -1."""
    nb, G, W, R = case["L"] // case["block"], case["n_global_blocks"], case["window_blocks"], case["n_random_blocks"]
    table = []
    for b in range(G, nb):
        own = set(range(max(0, b - W), min(nb, b + W + 1))) | set(range(G))
        key, a, want = _mix64(seed + 3 + _GOLD * (b + 1)), 0, len(own) + R
        while len(own) < want:
            own.add(_mix64(key + _GOLD * (a + 1)) % nb)
            a += 1
        table.append(sorted(own) + [-1] * (2 * W + 1 + G + R - len(own)))
    return torch.tensor(table, device="cuda")


def _bigbird(case, seed, Q, K, V, scale):
    H, L, d = Q.shape
    B, G = case["block"], case["n_global_blocks"]
    O = torch.empty((H, L, d), dtype=torch.float64, device="cuda")
    lse = torch.empty((H, L), dtype=torch.float64, device="cuda")
    table = _bigbird_blocks(case, seed)
    keys = (table.clamp(min=0)[:, :, None] * B + torch.arange(B, device="cuda")).flatten(1)
    ok = (table >= 0)[:, None, :, None].expand(-1, B, -1, B).flatten(2)
    step = max(1, int(1.5e8 / (H * B * keys.shape[1])))
    for b0 in range(0, keys.shape[0], step):
        b1 = min(keys.shape[0], b0 + step)
        r = slice((G + b0) * B, (G + b1) * B)
        k = keys[b0:b1]
        o, l = _softmax_v(Q[:, r].double().reshape(H, b1 - b0, B, d), K[:, k].double(), V[:, k].double(),
                          ok[None, b0:b1], scale)
        O[:, r], lse[:, r] = o.reshape(H, -1, d), l.reshape(H, -1)
    for h in range(H):      # the global rows attend every key
        for r0 in range(0, G * B, 64):
            n = min(64, G * B - r0)
            o, l = _softmax_v(Q[h, r0:r0 + n].double(), K[h].double(), V[h].double(),
                              torch.ones((n, 1), dtype=torch.bool, device="cuda"), scale)
            O[h, r0:r0 + n], lse[h, r0:r0 + n] = o, l
    return O, lse


def exact(case, seed):
    H, L, d, scale, kind = case["H"], case["L"], case["d"], _scale(case), case["mask"]
    Q, K, V = _qkv(case, seed)
    if kind in ("random", "bigbird_model"):
        O = torch.empty((H, L, d), dtype=torch.float64, device="cuda")
        lse = torch.empty((H, L), dtype=torch.float64, device="cuda")
        for r0, ok in _random_rows(case, seed):
            if kind == "bigbird_model":
                ok = ok | _longformer_rows(case, r0, ok.shape[0])
            _dense_rows(Q, K, V, ok, r0, O, lse, scale)
    elif kind == "bigbird":
        O, lse = _bigbird(case, seed, Q, K, V, scale)
    elif kind == "global_local":
        g = min(case["n_global"], L)
        O, lse = _band(Q, K, V, case["window"], scale, extra=g)
        ok = torch.ones((g, 1), dtype=torch.bool, device="cuda")
        for h in range(H):
            _dense_rows(Q[h:h + 1], K[h:h + 1], V[h:h + 1], ok, 0, O[h:h + 1], lse[h:h + 1], scale)
    elif kind == "dilated_2d":
        b, s = case["block"], case["stride"]
        O = torch.zeros((H, L, d), dtype=torch.float64, device="cuda")
        lse = torch.full((H, L), -math.inf, dtype=torch.float64, device="cuda")
        for b0 in range(0, L, b):
            r = slice(b0, min(L, b0 + b), s)
            ok = torch.ones((1, 1), dtype=torch.bool, device="cuda")
            O[:, r], lse[:, r] = _softmax_v(Q[:, r].double(), K[:, r].double(), V[:, r].double(), ok, scale)
    else:
        s = case.get("stride", 1)
        O = torch.empty((H, L, d), dtype=torch.float64, device="cuda")
        lse = torch.empty((H, L), dtype=torch.float64, device="cuda")
        for r in range(s):
            O[:, r::s], lse[:, r::s] = _band(Q[:, r::s], K[:, r::s], V[:, r::s], case["window"], scale)
    if case["op"] == "step":
        return {"O": O, "row_ptr": None, "col_idx": None}
    return {"O": O, "lse": lse} if case["op"] in ("compose", "static") else {"O": O}
