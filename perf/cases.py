"""Performance cases of the ReLU-sparse FFN layer: what a program that uses the library has it do.

A case is a dict of plain values. `prepare` makes what such a program holds before the call
(activations, weights, the weight copies it keeps, buffers and workspaces), `run` makes one
pass through the library's entry points, `exact` computes the same outputs in float64 with
plain torch, and `work` states the bytes and operations the pass cannot do without.

Inputs follow the recipe of the repository's workloads: X ~ N(0, 1), weights ~ N(0, 0.02^2),
and a per-token shift of the pattern-deciding projection that makes every hidden unit active
with probability 1 - sparsity (or gives each token its own active count, log-normal with a
heavy tail), or a constant bias per hidden unit.
"""
from __future__ import annotations

import math

import torch

from paper_2603_23198_amd import binding as b

SIGMA_W = 0.02  # standard deviation of the weights
LAMBDA_L1 = 2e-5  # L1 coefficient of the training steps
BIAS_SIGMAS = 2.5  # the biased fp32 layer: bias = -2.5 standard deviations of the pre-activation


def _case(path, **kw):
    """A case with the defaults of an ordinary one.

    path: "forward" (one sfl_ffn_forward), "train" (forward, the dead-unit record for the
    non-gated layer, and backward) or "pack" (sfl_pack_twell of fp32 pre-activations).
    copies: the program keeps the transposed and slice-major weight copies beside the weights
    (inference, and the micro-batches of one optimizer step); without them it hands over the
    plain weights, as in the first pass after an update.
    capacity: rows of the dense backup, 0 for one per token."""
    c = dict(path=path, dtype="bf16", gated=False, T=1, d=512, f=1024, sparsity=0.99, rows="uniform", ell_width=64,
             tile_cols=256, tile_slots=32, packed32=False, capacity=0, copies=True)
    c.update(kw)
    return c


def listed():
    return [
        # The small fp32 layer with a per-unit bias: the exact-precision path, launch bound.
        _case("forward", name="fp32_64_tokens", dtype="f32", T=64, d=256, f=1024, rows="bias", sparsity=0.9938,
              ell_width=32),
        # One sequence being decoded: one token through a 2048-wide layer.
        _case("forward", name="decode_1_token", T=1, d=2048, f=8192, ell_width=192),
        # A batch of 32 sequences being decoded through a gated 4096-wide layer.
        _case("forward", name="decode_gated_32_tokens", gated=True, T=32, d=4096, f=14336, sparsity=0.995,
              ell_width=128),
        # A prompt chunk of odd length through a gated 2048-wide layer (f not a multiple of 512).
        _case("forward", name="chunk_gated_509_tokens", gated=True, T=509, d=2048, f=5632, sparsity=0.995,
              ell_width=64),
        # A prompt chunk, or one GPU's share of the tokens when eight split the batch, in the
        # packed 32-bit storage of the activations.
        _case("forward", name="chunk_1024_tokens_packed32", T=1024, d=4096, f=16384, ell_width=256, tile_slots=31,
              packed32=True),
        # Heavy-tailed active counts: every sixth token is a dense-backup row.
        _case("forward", name="lognormal_4096_tokens", T=4096, d=2048, f=8192, rows="lognormal", ell_width=128),
        # The library's benchmark: a full prefill batch at 99 %.
        _case("forward", name="prefill_8192_tokens", T=8192, d=4096, f=16384, ell_width=256),
        # Weak sparsity, as before the L1 term has done its work: the dense fallback decides.
        _case("forward", name="prefill_95_percent", T=8192, d=4096, f=16384, sparsity=0.95, ell_width=1024,
              tile_slots=48),
        # A full prefill batch of the gated layer.
        _case("forward", name="prefill_gated_8192_tokens", gated=True, T=8192, d=4096, f=14336, sparsity=0.995,
              ell_width=128),
        # One micro-batch of training: forward, the record of active units, backward.
        _case("train", name="train_16384_tokens", T=16384, d=4096, f=16384, ell_width=256),
        # The gated layer's first micro-batch after an update (no weight copies yet), the dense
        # backup sized to an eighth of the tokens.
        _case("train", name="train_gated_8192_tokens", gated=True, T=8192, d=4096, f=14336, sparsity=0.995,
              ell_width=128, capacity=1024, copies=False),
        # Packing pre-activations that another program computed, ragged in both directions.
        _case("pack", name="pack_4001_tokens", T=4001, d=64, f=5600, sparsity=0.99, ell_width=128),
    ]


def _ell_width(f, sparsity):
    """Six standard deviations above the mean active count, in steps of 64."""
    mean, sd = f * (1 - sparsity), math.sqrt(f * sparsity * (1 - sparsity))
    return int(min(max(64, math.ceil((mean + 6 * sd) / 64) * 64), math.ceil(f / 64) * 64))


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward"] * 4 + ["gated"] * 3 + ["f32", "train", "train_gated", "pack"])
    if kind == "pack":
        f, sparsity = _log_int(rng, 100, 16384), rng.choice([0.95, 0.99, 0.995])
        return _case("pack", T=_log_int(rng, 1, 8192), d=64, f=f, sparsity=sparsity, ell_width=_ell_width(f, sparsity),
                     tile_slots=48 if sparsity < 0.97 else 32, dtype=rng.choice(["bf16", "bf16", "f32"]))
    if kind == "f32":
        return _case("forward", dtype="f32", T=_log_int(rng, 1, 512), d=2 * _log_int(rng, 32, 512),
                     f=_log_int(rng, 256, 4096), rows="bias", sparsity=0.9938, ell_width=64)
    train, gated = kind.startswith("train"), kind in ("gated", "train_gated")
    T = _log_int(rng, 256, 8192) if train else _log_int(rng, 1, 8192)
    d = 512 * rng.randint(1, 8)
    if kind == "forward" and rng.random() < 0.25:
        d = 64 * rng.randint(4, 64)
    # hidden layers are a few times wider than the model
    f = 64 * _log_int(rng, 16 if d <= 2048 else 116, 224 if gated else 256)
    sparsity = rng.choice([0.99, 0.995, 0.998, 0.999])
    c = _case("train" if train else "forward", gated=gated, T=T, d=d, f=f, sparsity=sparsity,
              ell_width=_ell_width(f, sparsity), copies=rng.random() < 0.75)
    if train:
        c["capacity"] = rng.choice([0, max(1, T // 8)])
        return c
    if kind == "forward" and rng.random() < 0.2:
        c.update(sparsity=0.95, tile_slots=48, ell_width=_ell_width(f, 0.95))
    elif f >= 4096 and rng.random() < 0.2:
        c.update(rows="lognormal", sparsity=0.99, ell_width=128)
    elif rng.random() < 0.25:
        c.update(packed32=True, tile_slots=31)
    elif rng.random() < 0.15:
        c.update(tile_cols=128, tile_slots=24)
    return c


# ---- inputs ---------------------------------------------------------------------------------

def _inputs(case, seed):
    """The case's tensors on the GPU, from the seed alone."""
    T, d, f = case["T"], case["d"], case["f"]
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + T * 31 + d * 7 + f)
    act = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(shape, std, dtype):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(dtype)

    if case["path"] == "pack":
        Z = normal((T, f), 1.0, torch.float32)
        Z -= float(torch.special.ndtri(torch.tensor(case["sparsity"], dtype=torch.float64)))
        return dict(Z=Z)
    s = dict(X=normal((T, d), 1.0, act), W_up=normal((d, f), SIGMA_W, act), W_down=normal((f, d), SIGMA_W, act),
             W_gate=normal((d, f), SIGMA_W, act) if case["gated"] else None, bias_f=None, shift_t=None)
    if case["path"] == "train":
        s["dY"] = normal((T, d), 1.0, act)
    if case["rows"] == "bias":
        s["bias_f"] = torch.full((f,), -BIAS_SIGMAS * SIGMA_W * math.sqrt(d), device="cuda", dtype=torch.float32)
        return s
    sparsity = torch.full((T,), case["sparsity"], device="cuda", dtype=torch.float64)
    if case["rows"] == "lognormal":
        mean, sigma = f * (1 - case["sparsity"]), 0.8
        n = torch.randn((T,), generator=g, device="cuda", dtype=torch.float64)
        n = (n * sigma + (math.log(mean) - sigma * sigma / 2)).exp().clamp_(1, 12 * mean)
        sparsity = 1 - n / f
    s["shift_t"] = (-SIGMA_W * s["X"].double().norm(dim=1) * torch.special.ndtri(sparsity)).float()
    return s


def _bytes(n):
    return torch.empty(max(1, n), dtype=torch.uint8, device="cuda")


def _copies(s):
    """The weight copies an inference program keeps beside the weights."""
    def transposed(W):
        out = torch.empty((W.shape[1], W.shape[0]), dtype=W.dtype, device="cuda")
        b.sfl_transpose(W, out)
        return out

    def slices(W):
        out = torch.empty_like(W)
        b.sfl_pack_down_weights(W, out)
        return out

    k = dict(W_upT=transposed(s["W_up"]), W_downT=transposed(s["W_down"]))
    if s["W_up"].shape[0] % 512 == 0:
        k["W_down_packed"], k["W_up_packed"] = slices(s["W_down"]), slices(k["W_upT"])
    if s["W_gate"] is not None:
        k["W_gateT"] = transposed(s["W_gate"])
        k["W_gate_packed"] = slices(k["W_gateT"])
    return k


def prepare(case, seed):
    T, d, f = case["T"], case["d"], case["f"]
    cfg = b.make_cfg(tile_cols=case["tile_cols"], tile_slots=case["tile_slots"], ell_width=case["ell_width"],
                     ovf_capacity=case["capacity"], layout=b.SFL_TWELL_PACKED32 if case["packed32"] else 0)
    s = _inputs(case, seed)
    s.update(case=case, cfg=cfg, bufs=b.alloc_twell(T, f, case["dtype"], cfg, with_dense=case["path"] != "pack"),
             stats=b.alloc_stats())
    if case["path"] == "pack":
        for t in s["bufs"].values():  # slots beyond a tile's count stay as they were
            if t is not None:
                t.zero_()
        return s
    copies = _copies(s) if case["copies"] and case["dtype"] == "bf16" else {}
    s["copies"] = copies
    s["Y"] = torch.empty_like(s["X"])
    fwd = {k: v for k, v in copies.items() if k != "W_gate_packed"}
    kw = dict(Y=s["Y"], bufs=s["bufs"], W_gate=s["W_gate"], bias_f=s["bias_f"], shift_t=s["shift_t"],
              stats=s["stats"], **fwd)
    s["fwd_ws"] = _bytes(b.sfl_workspace_size(b.ffn_args(s["X"], s["W_up"], s["W_down"], cfg, **kw)))
    s["fwd"] = b.ffn_args(s["X"], s["W_up"], s["W_down"], cfg, workspace=s["fwd_ws"], **kw)
    if case["path"] == "train":
        s["dX"] = torch.empty_like(s["X"])
        for n in ("W_up", "W_down") + (("W_gate",) if case["gated"] else ()):
            s["d" + n] = torch.empty(s[n].shape, dtype=torch.float32, device="cuda")
        bwd = {k: v for k, v in copies.items() if k != "W_downT"}
        if case["gated"]:
            bwd.update(W_gate=s["W_gate"], dW_gate=s["dW_gate"], bias_f=s["bias_f"], shift_t=s["shift_t"])
        pos = (s["X"], s["W_up"], s["W_down"], s["dY"], cfg, s["bufs"], LAMBDA_L1, s["dX"], s["dW_up"], s["dW_down"])
        s["bwd_ws"] = _bytes(b.sfl_workspace_size(b.bwd_args(*pos, **bwd), 1))
        s["bwd"] = b.bwd_args(*pos, workspace=s["bwd_ws"], **bwd)
        s["last_active"] = torch.zeros((f,), dtype=torch.int64, device="cuda")
    return s


def run(s):
    case, T = s["case"], s["case"]["T"]
    if case["path"] == "pack":
        b.sfl_pack_twell(s["Z"], case["dtype"], s["cfg"], s["bufs"], stats=s["stats"])
        return {n: s["bufs"][n] for n in ("val", "idx", "cnt", "row_nnz", "row_ovf", "n_ovf", "ell_val", "ell_idx")}
    b.sfl_ffn_forward(s["fwd"])
    out = dict(Y=s["Y"], row_nnz=s["bufs"]["row_nnz"][:T], l1=s["stats"].view(torch.float64)[3:4])
    if case["path"] == "train":
        if not case["gated"]:
            b.sfl_track_active_units(s["bufs"], T, case["f"], case["dtype"], s["cfg"], 1, s["last_active"])
            out["last_active"] = s["last_active"]
        b.sfl_ffn_backward(s["bwd"])
        out.update({n: s[n] for n in ("dX", "dW_up", "dW_down") + (("dW_gate",) if case["gated"] else ())})
    return out


# ---- what a pass needs, and what it has to give ---------------------------------------------

def work(case):
    T, d, f = case["T"], case["d"], case["f"]
    es = 2 if case["dtype"] == "bf16" else 4
    if case["path"] == "pack":
        tiles = -(-f // case["tile_cols"])
        nnz = T * f * (1 - case["sparsity"])
        return {"bytes": T * f * 4 + T * tiles * 4 + 2 * nnz * (es + 2) + 5 * T, "flops": T * f}
    mats = 3 if case["gated"] else 2
    active = 1 - case["sparsity"]
    nnz = T * f * active
    weights = d * f * es
    # the pattern-deciding projection reads its whole matrix; the others only the rows of units
    # that some token activates
    touched = 1 - (1 - active) ** T
    fwd_bytes = 2 * T * d * es + weights * (1 + (mats - 1) * touched)
    fwd_flops = 2 * T * d * f + 2 * nnz * d * (mats - 1)
    if case["path"] == "forward":
        return {"bytes": fwd_bytes, "flops": fwd_flops}
    # backward: dh at the pattern and dX (one product per input weight matrix), one product per
    # weight gradient (fp32, written whole), and the recomputed up projection of the gated layer
    products = 1 + (mats - 1) + mats + (1 if case["gated"] else 0)
    return {"bytes": fwd_bytes + 3 * T * d * es + mats * (weights * touched + d * f * 4),
            "flops": fwd_flops + 2 * nnz * d * products}


def tolerance(case):
    if case["path"] == "pack":
        return "exact"
    if case["dtype"] == "f32":
        # against float64: 1.6e-6 in Y (few active units, each with a pre-activation that is a
        # small difference); another order of the sums moves it by about as much. An active
        # count differs only where a pre-activation is within rounding of zero.
        return {"rel": 6e-6, "max": 1e-4, "differ": 0.002}
    if case["path"] == "train":
        # A pre-activation within rounding of zero may be active in one order of the sums and not
        # in another (a few per 1e8), which moves single elements of a unit's weight gradient.
        return {"rel": 1e-2, "max": 0.9, "differ": 0.002}
    # bf16 activations and output: 2e-3 to 3e-3 against float64
    return {"rel": 1e-2, "max": 0.1, "differ": 0.002}


def exact(case, seed):
    if case["path"] == "pack":
        return None  # whole numbers and bytes
    s = _inputs(case, seed)
    T, f = case["T"], case["f"]
    X, Wu, Wd = s["X"].double(), s["W_up"].double(), s["W_down"].double()
    Wg = s["W_gate"].double() if case["gated"] else None
    Z = X @ (Wg if case["gated"] else Wu)
    if s["bias_f"] is not None:
        Z += s["bias_f"].double()
    if s["shift_t"] is not None:
        Z += s["shift_t"].double()[:, None]
    on = Z > 0
    G = Z.clamp_(min=0)
    U = X @ Wu if case["gated"] else None
    H = G * U if case["gated"] else G
    out = dict(Y=H @ Wd, row_nnz=None, l1=H.abs().sum().reshape(1))
    if case["path"] == "train":
        dY = s["dY"].double()
        dH = dY @ Wd.t()
        dH += (LAMBDA_L1 / (T * f)) * H.sign()
        dH *= on
        if case["gated"]:
            dU, dG = dH * G, dH * U
            out.update(dX=dU @ Wu.t() + dG @ Wg.t(), dW_up=X.t() @ dU, dW_down=H.t() @ dY, dW_gate=X.t() @ dG)
        else:
            out.update(last_active=None, dX=dH @ Wu.t(), dW_up=X.t() @ dH, dW_down=H.t() @ dY)
    return out
