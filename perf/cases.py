"""Performance cases: what programs have this library do, through its Python entry points.

Every case is a plain dict.  `kind` names the call sequence:
    decode    one token per sequence against the carried state (la_decode_step)
    prefill   a prompt, or a piece of one, with the state carried in and out (la_fwd_state)
    train     la_fwd and la_bwd of one attention layer, contiguous [B, H, n, d] tensors
    strided   the same on [B, n, H, d] projection outputs (la_fwd_strided, la_bwd_strided)
    swish     the same with the query / key activation fused in (la_fwd_swish, la_bwd_swish)
    lrpe      an LRPE-d layer: rotation of Q and K, wide attention, and both backward
    gate      the gated SRMSNorm output stage, forward and backward
"""
from __future__ import annotations

import math

import torch

from paper_2405_17381_amd import binding, synth

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(kind, B, H, n, d, dtype="bf16", decay="geometric", name=None):
    c = {"kind": kind, "B": B, "H": H, "n": n, "d": d, "dtype": dtype, "decay": decay}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # token-by-token generation for a batch of 8 requests on a 32-head layer: the smallest call
        _case("decode", 8, 32, 1, 128, name="decode"),
        # one 1000-token prompt (ragged) entering generation on a 16-head layer
        _case("prefill", 1, 16, 1000, 128, name="prefill"),
        # the smallest training call, in fp32 with 64 features (workload c1 of synth.py): latency
        _case("train", 1, 2, 256, 64, "f32", "ones", name="train_c1"),
        # a small 64-feature layer at 2048 tokens (workload c2)
        _case("train", 4, 16, 2048, 64, "bf16", "exponential", name="train_c2"),
        # the two ends of the 65536-token sweep: many short sequences, one long one (workload c3)
        _case("train", 32, 16, 2048, 128, name="train_2k"),
        _case("train", 1, 16, 65536, 128, name="train_64k"),
        # a 32-head layer, batch 8, 4096 tokens (workload c4)
        _case("train", 8, 32, 4096, 128, name="train_c4"),
        # training in fp32
        _case("train", 8, 16, 2048, 128, "f32", name="train_f32"),
        # projection outputs used where they lie, [B, n, H, d], length not a multiple of any tile
        _case("strided", 2, 16, 5003, 128, name="token_major"),
        # gated linear attention with the activation inside the kernels
        _case("swish", 4, 16, 8192, 128, name="swish"),
        # the first layer of the model: LRPE-d on one long sequence
        _case("lrpe", 1, 16, 65536, 128, name="lrpe"),
        # the output stage of a layer on the sweep's 65536 tokens
        _case("gate", 1, 16, 65536, 128, name="gate"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "prefill", "train", "train", "train", "strided", "swish", "lrpe", "gate"])
    d = rng.choice([64, 128, 128])
    decay = rng.choice(["geometric", "exponential", "ones", "half"])
    H = rng.choice([1, 2, 3, 5, 8, 12, 16, 16, 32])
    if kind == "decode":
        return _case(kind, _log(rng, 1, 128), H, 1, d, rng.choice(["bf16", "bf16", "f32"]), decay)
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    # elements of one [B, H, n, d] tensor, then how they are split over batch and length
    top = {"prefill": 1 << 24, "lrpe": 1 << 25}.get(kind, 1 << 26)
    if dtype == "f32":
        top >>= 2
    tokens = max(16, _log(rng, 1 << 15, top) // (H * d))
    n = min(tokens, _log(rng, 16, 131072))
    B = 1 if kind == "prefill" else max(1, min(64, tokens // n))
    return _case(kind, B, H, n, d, dtype, decay)


def _lambdas(case):
    H = case["H"]
    if case["decay"] == "geometric":
        lam = synth.lambda_geometric(0.9, 0.9999, H)
    elif case["decay"] == "exponential":
        lam = synth.lambda_exp_schedule(H)
    elif case["decay"] == "ones":
        lam = [1.0, 0.99] * (H // 2) + [1.0] * (H % 2)
    else:       # half of the heads do not decay
        lam = [1.0] * (H - H // 2) + synth.lambda_geometric(0.95, 0.9999, H // 2)[: H // 2]
    return [float(torch.tensor(x, dtype=torch.float32)) for x in lam]


def _inputs(case, seed):
    """Tensors by name, in the case's dtype, contiguous [B, H, n, d] (decode: [B, H, d])."""
    B, H, n, d = case["B"], case["H"], case["n"], case["d"]
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)

    x = {}
    kind, s = case["kind"], 1.0 / math.sqrt(d)
    if kind == "gate":
        for k in ("O", "U", "dY"):
            x[k] = normal(B, H, n, d)
    elif kind == "decode":
        for k in ("Q", "K", "V"):
            x[k] = normal(B, H, d) * s
    else:
        for k in ("Q", "K", "V"):
            x[k] = normal(B, H, n, d)
            # the activated projections are of order one before the activation; V keeps O there
            x[k] *= s if kind != "swish" else (1.0 / d if k == "V" else 1.0)
        if kind != "prefill":
            x["dO"] = normal(B, H, n, d)
    x = {k: v.to(_DT[case["dtype"]]) for k, v in x.items()}
    if kind in ("decode", "prefill"):
        x["kv"] = normal(B, H, d, d) * s
    if kind == "lrpe":
        x["theta"] = torch.rand((H, d), generator=gen, device="cuda", dtype=torch.float32)
    return x


def prepare(case, seed):
    B, H, n, d = case["B"], case["H"], case["n"], case["d"]
    dtype, kind = _DT[case["dtype"]], case["kind"]
    dt = binding.LA_BF16 if case["dtype"] == "bf16" else binding.LA_F32
    s = {"kind": kind, "lam": _lambdas(case)}
    s.update(_inputs(case, seed))

    def new(*shape):
        return torch.empty(shape, device="cuda", dtype=dtype)

    def scratch(nbytes):
        return torch.empty(max(256, nbytes), device="cuda", dtype=torch.uint8)

    if kind == "decode":
        s["o"] = new(B, H, d)
    elif kind == "gate":
        for k in ("Y", "gO", "gU"):
            s[k] = new(B, H, n, d)
    elif kind == "prefill":
        s["O"] = new(B, H, n, d)
        s["kv_out"] = torch.empty((B, H, d, d), device="cuda", dtype=torch.float32)
        s["ws"] = scratch(binding.la_workspace_bytes(B, H, n, d, dt, False))
    else:
        if kind == "strided":
            for k in ("Q", "K", "V", "dO"):
                s[k] = s[k].transpose(1, 2).contiguous().transpose(1, 2)
            for k in ("O", "dQ", "dK", "dV"):
                s[k] = new(B, n, H, d).transpose(1, 2)
        else:
            for k in ("O", "dQ", "dK", "dV"):
                s[k] = new(B, H, n, d)
        s["ws"] = scratch(binding.la_workspace_bytes(B, H, n, d, dt, True))
        if kind == "lrpe":
            for k in ("Qw", "Kw", "dQw", "dKw"):
                s[k] = new(B, H, n, 2 * d)
            s["dtheta"] = torch.empty((H, d), device="cuda", dtype=torch.float32)
            s["lws"] = scratch(binding.la_lrpe_workspace_bytes(B, H, n, d))
    return s


def run(s):
    kind, lam = s["kind"], s["lam"]
    if kind == "decode":
        binding.la_decode_step(s["Q"], s["K"], s["V"], lam, s["kv"], o=s["o"])
        return s["o"], s["kv"]
    if kind == "prefill":
        binding.la_fwd_state(s["Q"], s["K"], s["V"], lam, kv_in=s["kv"], kv_out=s["kv_out"], O=s["O"],
                             workspace=s["ws"])
        return s["O"], s["kv_out"]
    if kind == "gate":
        binding.la_gate_norm_fwd(s["O"], s["U"], 0.0, Y=s["Y"])
        binding.la_gate_norm_bwd(s["O"], s["U"], s["dY"], 0.0, dO=s["gO"], dU=s["gU"])
        return s["Y"], s["gO"], s["gU"]
    Q, K, V, dO, ws = s["Q"], s["K"], s["V"], s["dO"], s["ws"]
    O, dQ, dK, dV = s["O"], s["dQ"], s["dK"], s["dV"]
    if kind == "train":
        binding.la_fwd(Q, K, V, lam, O=O, workspace=ws)
        binding.la_bwd(Q, K, V, lam, dO, dQ=dQ, dK=dK, dV=dV, workspace=ws)
    elif kind == "strided":
        binding.la_fwd_strided(Q, K, V, lam, O=O, workspace=ws)
        binding.la_bwd_strided(Q, K, V, lam, dO, dQ=dQ, dK=dK, dV=dV, workspace=ws)
    elif kind == "swish":
        binding.la_fwd_swish(Q, K, V, lam, O=O, workspace=ws)
        binding.la_bwd_swish(Q, K, V, lam, dO, dQp=dQ, dKp=dK, dV=dV, workspace=ws)
    else:
        th, Qw, Kw, lws = s["theta"], s["Qw"], s["Kw"], s["lws"]
        binding.la_lrpe_rotate_fwd(Q, th, Xw=Qw)
        binding.la_lrpe_rotate_fwd(K, th, Xw=Kw)
        binding.la_fwd_wide(Qw, Kw, V, lam, O=O, workspace=ws)
        binding.la_bwd_wide(Qw, Kw, V, lam, dO, dQw=s["dQw"], dKw=s["dKw"], dV=dV, workspace=ws)
        binding.la_lrpe_rotate_bwd(Q, th, s["dQw"], dX=dQ, dtheta=s["dtheta"], workspace=lws)
        binding.la_lrpe_rotate_bwd(K, th, s["dKw"], dX=dK, dtheta=s["dtheta"], accumulate=True, workspace=lws)
        return O, dQ, dK, dV, s["dtheta"]
    return O, dQ, dK, dV


def work(case):
    B, H, n, d, kind = case["B"], case["H"], case["n"], case["d"], case["kind"]
    e = 2 if case["dtype"] == "bf16" else 4
    rows = B * H * n
    t = rows * d * e                            # one [B, H, n, d] tensor
    state = B * H * d * d * 4
    if kind == "decode":
        return {"bytes": 2 * state + 4 * t, "flops": 5 * B * H * d * d}
    if kind == "prefill":
        return {"bytes": 2 * state + 4 * t, "flops": rows * 8 * d * d}
    if kind == "gate":                          # forward 2 in, 1 out; backward 3 in, 2 out
        return {"bytes": 8 * t, "flops": rows * d * 15}
    # attention: forward 3 in, 1 out; backward 4 in, 3 out
    if kind == "lrpe":
        # wide forward (2 + 2 + 1 in, 1 out) and backward (2 + 2 + 1 + 1 in, 2 + 2 + 1 out), and per
        # tensor of two the rotation (1 in, 2 out) and its backward (1 + 2 in, 1 out)
        return {"bytes": (6 + 11 + 2 * 3 + 2 * 4) * t, "flops": 2 * rows * 30 * d * d}
    return {"bytes": 11 * t, "flops": rows * 30 * d * d}


def tolerance(case):
    # relative 2-norm, about four times what the kernels show against 64-bit arithmetic
    # (fp32 5e-7; bf16 results 1.7e-3 to 2.9e-3, activated ones 3.7e-3, LRPE-d's 4.1e-3)
    if case["kind"] == "lrpe" and case["n"] > 8192:
        # theta's gradient: a sum over all rows, weighted by the row number, whose terms cancel;
        # on 65536 rows the roundings of its bf16 inputs alone come to 3.3e-2
        return {"rel": 0.1 if case["dtype"] == "bf16" else 4e-5}
    if case["dtype"] == "f32":
        return {"rel": 2e-5 if case["kind"] == "lrpe" else 4e-6}
    return {"rel": {"decode": 8e-3, "gate": 8e-3, "swish": 1.5e-2, "lrpe": 2.5e-2}.get(case["kind"], 1.2e-2)}


# ---- the same results in 64-bit torch ------------------------------------------------------------

def _scan64(A, Bm, C, lam, reverse=False, st=None):
    """Out[t] = sum_{s <= t} lambda^(t-s) (A[t] . Bm[s]) C[s] (reverse: s >= t), 128 tokens at a time;
    returns Out and the state sum_s lambda^(n-1-s) Bm[s] C[s]^T."""
    if reverse:
        out, st = _scan64(A.flip(2), Bm.flip(2), C.flip(2), lam)
        return out.flip(2), st
    B, H, n, _ = A.shape
    dev = A.device
    lg = torch.log(torch.tensor(lam, dtype=torch.float64, device=dev)).view(1, H, 1, 1)
    if st is None:
        st = torch.zeros((B, H, Bm.shape[3], C.shape[3]), dtype=torch.float64, device=dev)
    out = torch.empty((B, H, n, C.shape[3]), dtype=torch.float64, device=dev)
    for t0 in range(0, n, 128):
        m = min(128, n - t0)
        a, b, c = (x[:, :, t0:t0 + m].to(torch.float64).contiguous() for x in (A, Bm, C))
        r = torch.arange(m, dtype=torch.float64, device=dev)
        dist = r.view(m, 1) - r.view(1, m)
        mask = torch.where(dist >= 0, torch.exp(dist.clamp(min=0) * lg), torch.zeros((), dtype=torch.float64, device=dev))
        scores = (a @ b.transpose(2, 3).contiguous()) * mask
        out[:, :, t0:t0 + m] = scores @ c + (a @ st) * torch.exp((r.view(m, 1) + 1) * lg)
        w = torch.exp((m - 1 - r.view(m, 1)) * lg)
        st = torch.exp(m * lg) * st + (b * w).transpose(2, 3).contiguous() @ c
    return out, st



def exact(case, seed):
    x = _inputs(case, seed)
    lam, kind, d = _lambdas(case), case["kind"], case["d"]
    f = {k: v.to(torch.float64) for k, v in x.items()}
    if kind == "decode":
        l = torch.tensor(lam, dtype=torch.float64, device="cuda").view(1, -1, 1, 1)
        kv = l * f["kv"] + f["K"].unsqueeze(3) * f["V"].unsqueeze(2)
        return (f["Q"].unsqueeze(3) * kv).sum(2), kv
    if kind == "prefill":
        return _scan64(f["Q"], f["K"], f["V"], lam, st=f["kv"])
    if kind == "gate":
        O, U, g = f["O"], f["U"], f["dY"]
        r = O.square().mean(dim=(1, 3), keepdim=True).sqrt()
        dn = g * U
        return O / r * U, dn / r - O * (dn * O).mean(dim=(1, 3), keepdim=True) / r ** 3, g * O / r
    Q, K, V, dO = f["Q"], f["K"], f["V"], f["dO"]
    if kind == "swish":
        sq, sk = torch.sigmoid(Q), torch.sigmoid(K)
        gq, gk = sq * (1 + Q * (1 - sq)), sk * (1 + K * (1 - sk))
        Q, K = Q * sq, K * sk
    if kind == "lrpe":
        t = torch.arange(case["n"], dtype=torch.float64, device="cuda").view(1, 1, -1, 1)
        ang = t * f["theta"].view(1, case["H"], 1, d)
        cs, sn = torch.cos(ang), torch.sin(ang)
        del ang
        q0, k0 = Q, K
        Q, K = torch.cat((Q * cs, Q * sn), 3), torch.cat((K * cs, K * sn), 3)
    O = _scan64(Q, K, V, lam)[0]
    dQ = _scan64(dO, V, K, lam)[0]
    dK = _scan64(V, dO, Q, lam, reverse=True)[0]
    dV = _scan64(K, Q, dO, lam, reverse=True)[0]
    if kind == "swish":
        return O, dQ * gq, dK * gk, dV
    if kind == "lrpe":
        res, dth = [], 0.0
        for x0, g in ((q0, dQ), (k0, dK)):
            gc, gs = g[..., :d], g[..., d:]
            res.append(gc * cs + gs * sn)
            dth = dth + (t * x0 * (gs * cs - gc * sn)).sum(dim=(0, 2))
        return O, res[0], res[1], dV, dth
    return O, dQ, dK, dV
