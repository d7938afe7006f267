"""The work this library is used for, as cases that can be timed and checked one by one.

A case is a dict of plain values. `kind` says which entry points it goes through:

  fwd        fwd                                   inference, or the first half of a step
  train      attention (autograd) and its backward a training step of one layer, fp32 upstream gradient
  fwdbwd     fwd, bwd                              a training step through the explicit entry points
  ds         fwd, bwd(store_ds=True)               the same with the stored-dS backward, workspace kept
  segments   fwd per key segment, merge, bwd per segment with accumulate_dq
  layouts    the four layout copies around a Ulysses all-to-all (bf16 Q, K, V in; fp32 O out)
  channels   agg_fwd, agg_bwd                      the channel aggregation of one layer

Sizes are the shards of the paper's models: heads of 64, 72, 128 and 160, 512 to 1,048,576 tokens,
whole batches of short sequences down to one head of a long one.
"""
import math

import torch

import paper_2405_15780_amd as va


def listed():
    return [
        # one head over a 32x32 patch grid: the smallest call, launch and latency
        _attn("head_1k_fwd", "fwd", 1, 1, 1024, 64),
        # ViT-Base at 16K tokens per step in 1,024-token images: many short sequences
        _attn("vit_base_1k_train", "train", 16, 16, 1024, 64),
        # 128x128 patches, two of ViT-5B's heads on this GPU: half a chip's worth of query blocks
        _attn("shard_16k_d128_train", "train", 1, 2, 16384, 128),
        # the same image as a whole ViT-Base block; head 0 has near one-hot rows
        _attn("block_16k_d64", "fwdbwd", 2, 16, 16384, 64, stress=8.0),
        # ViT-10B's heads of 72, an odd crop, operands sequence-major as an all-to-all leaves them
        _attn("seqmajor_20k_d72", "fwdbwd", 1, 2, 20001, 72, layout="bnhd"),
        # heads of 160 (width 2,560 over 16), a short odd sequence
        _attn("crop_5k_d160_train", "train", 1, 4, 5003, 160),
        # the stored-dS backward where its N x N workspace is small
        _attn("shard_32k_d128_ds", "ds", 1, 2, 32768, 128),
        # 368x512 patches (92 channels x 2,048), two heads: the paper-scale training shard
        _attn("shard_188k_d128", "fwdbwd", 1, 2, 188416, 128),
        # 1024x1024 patches, one head: the longest sequence, forward only
        _attn("million_fwd_d64", "fwd", 1, 1, 1048576, 64, sigma=0.5),
        # one worker's queries against four key segments in turn, then the backward of each
        dict(name="segments_16k_d128", kind="segments", B=1, H=2, Nq=4096, Nk=4096, S=4, d=128, sigma=1.0),
        # both all-to-alls of one attention on one of 8 ranks at 188,416 tokens
        dict(name="layouts_188k", kind="layouts", B=1, H=16, P=8, Nl=23552, d=64),
        # 92 channels of 2,048 patches, batch 4
        dict(name="channels_92", kind="channels", M=8192, H=16, C=92, d=64),
    ]


def _attn(name, kind, B, H, N, d, layout="bhnd", sigma=1.0, stress=1.0):
    return dict(name=name, kind=kind, B=B, H=H, N=N, d=d, layout=layout, sigma=sigma, stress=stress)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fwd", "fwd", "train", "train", "train", "fwdbwd", "fwdbwd", "ds", "segments", "layouts",
                       "channels", "channels"])
    if kind == "layouts":
        c = dict(kind=kind, B=rng.choice([1, 1, 2, 4]), H=rng.choice([8, 16, 32]), P=rng.choice([2, 4, 8]),
                 Nl=_log_int(rng, 256, 32768), d=rng.choice([64, 72, 128, 160]))
        while c["B"] * c["H"] * c["Nl"] * c["d"] > 8 * 23552 * 16 * 64:
            c["Nl"] = c["Nl"] // 2 + 1
        return c
    if kind == "channels":
        c = dict(kind=kind, M=_log_int(rng, 128, 8192), H=rng.choice([8, 16, 16]), C=rng.randint(3, 128),
                 d=rng.choice([64, 64, 128]))
        while c["M"] * c["H"] * c["C"] * c["d"] > 8192 * 16 * 92 * 64:
            c["M"] = c["M"] // 2 + 1
        return c
    d = rng.choice([64, 64, 72, 128, 128, 160, 160, 80, 96])
    B, H = rng.choice([1, 1, 1, 2, 4, 16]), rng.choice([1, 2, 2, 3, 4, 6, 8, 12, 16])
    if kind == "segments":
        c = dict(kind=kind, B=1, H=H, Nq=_log_int(rng, 512, 24000), Nk=_log_int(rng, 512, 24000),
                 S=rng.choice([2, 3, 4, 8]), d=d, sigma=1.0)
        while c["H"] * c["Nq"] * c["Nk"] * c["S"] * d > 4e12:
            c["Nq"] = c["Nq"] // 2 + 1
        return c
    N = _log_int(rng, 512, 200000)
    if rng.random() < 0.4:
        N = -(-N // 256) * 256
    most = 2e10 if kind == "ds" else 1.6e13 / (2.5 * d)
    while B * H * N * N > most:
        if B > 1:
            B //= 2
        elif H > 1:
            H = (H + 1) // 2
        else:
            N = N * 2 // 3
    c = _attn("", kind, B, H, N, d, layout=rng.choice(["bhnd", "bhnd", "bnhd"]))
    del c["name"]
    return c


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, sigma=1.0, dtype=torch.bfloat16):
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    return (x * sigma).to(dtype) if sigma != 1.0 else x.to(dtype)


def _qkv_do(case, seed):
    """q, k, v (bf16) and the upstream gradient (fp32 for the autograd step, else bf16), each [B, H, N, d]."""
    g = _gen(seed)
    B, H, N, d = case["B"], case["H"], case["N"], case["d"]
    out = []
    for i in range(4):
        if i == 3 and case["kind"] == "fwd":
            break
        dtype = torch.float32 if i == 3 and case["kind"] == "train" else torch.bfloat16
        if case["layout"] == "bnhd":
            x = _normal(g, (B, N, H, d), case["sigma"], dtype).transpose(1, 2)
        else:
            x = _normal(g, (B, H, N, d), case["sigma"], dtype)
        if i < 2 and case["stress"] != 1.0:
            x[:, 0] *= case["stress"]
        out.append(x)
    return out


def _segments(case, seed):
    g = _gen(seed)
    B, H, Nq, Nk, S, d = (case[x] for x in ("B", "H", "Nq", "Nk", "S", "d"))
    q, do = _normal(g, (B, H, Nq, d), case["sigma"]), _normal(g, (B, H, Nq, d), case["sigma"])
    ks = [_normal(g, (B, H, Nk, d), case["sigma"]) for _ in range(S)]
    vs = [_normal(g, (B, H, Nk, d), case["sigma"]) for _ in range(S)]
    return q, ks, vs, do


def _layouts(case, seed):
    g = _gen(seed)
    B, H, P, Nl, d = (case[x] for x in ("B", "H", "P", "Nl", "d"))
    qkv = [_normal(g, (B, Nl, H, d)) for _ in range(3)]
    return qkv, _normal(g, (B, H // P, P * Nl, d), dtype=torch.float32)


def _channels(case, seed):
    g = _gen(seed)
    M, H, C, d = (case[x] for x in ("M", "H", "C", "d"))
    return _normal(g, (H, d)), _normal(g, (M, H, C, d)), _normal(g, (M, H, C, d)), _normal(g, (M, H, d))


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "segments":
        s["x"] = _segments(case, seed)
    elif kind == "layouts":
        s["x"] = _layouts(case, seed)
    elif kind == "channels":
        s["x"] = _channels(case, seed)
    else:
        s["x"] = _qkv_do(case, seed)
        if kind == "train":
            for t in s["x"][:3]:
                t.requires_grad_()
        elif kind == "ds":  # the N x N workspace is allocated once and kept
            B, H, N, d = case["B"], case["H"], case["N"], case["d"]
            nbytes = va.workspace_bytes_kv(B, H, N, N, d, va.VITATTN_BWD_STORE_DS)
            s["workspace"] = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda")
    return s


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "fwd":
        o, lse = va.fwd(*state["x"])
        return {"o": o, "lse": lse}
    if kind == "train":
        q, k, v, do = state["x"]
        o = va.attention(q, k, v)
        dq, dk, dv = torch.autograd.grad(o, (q, k, v), do)
        return {"o": o.detach(), "dq": dq, "dk": dk, "dv": dv}
    if kind in ("fwdbwd", "ds"):
        q, k, v, do = state["x"]
        o, lse = va.fwd(q, k, v)
        dq, dk, dv = va.bwd(q, k, v, o, lse, do, workspace=state.get("workspace"), store_ds=kind == "ds")
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if kind == "segments":
        q, ks, vs, do = state["x"]
        o_parts = torch.empty((len(ks),) + tuple(q.shape), dtype=torch.float32, device=q.device)
        lse_parts = torch.empty(o_parts.shape[:-1], dtype=torch.float32, device=q.device)
        for i, (k, v) in enumerate(zip(ks, vs)):
            va.fwd(q, k, v, out=(o_parts[i], lse_parts[i]))
        o, lse = va.merge(o_parts, lse_parts)
        dq = torch.zeros_like(o)
        dks, dvs = [], []
        for k, v in zip(ks, vs):
            out = (dq, torch.empty(k.shape, dtype=torch.float32, device=k.device),
                   torch.empty(v.shape, dtype=torch.float32, device=v.device))
            va.bwd(q, k, v, o, lse, do, out=out, accumulate_dq=True)
            dks.append(out[1])
            dvs.append(out[2])
        return {"o": o, "lse": lse, "dq": dq, "dk": dks, "dv": dvs}
    if kind == "layouts":
        qkv, o = state["x"]
        sends = [va.ulysses_pack(x, case["P"]) for x in qkv]
        heads = [va.ulysses_unpack(x) for x in sends]
        back = va.ulysses_pack_out(o, case["P"])
        return {"send": sends, "heads": heads, "send_out": back, "out": va.ulysses_unpack_out(back)}
    q, k, v, do = state["x"]
    o, lse = va.agg_fwd(q, k, v)
    dq, dk, dv = va.agg_bwd(q, k, v, o, lse, do)
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


def work(case):
    kind, d = case["kind"], case["d"]
    if kind == "layouts":
        rows = case["B"] * case["H"] * case["Nl"]
        # three bf16 tensors through two copies each, one fp32 tensor through two
        return {"bytes": rows * d * (3 * 2 * 2 * 2 + 2 * 2 * 4), "flops": 0}
    if kind == "channels":
        n = case["M"] * case["H"]
        # forward: K, V in, O and LSE out; backward: K, V, O, dO, LSE in, dK, dV out
        return {"bytes": n * (case["C"] * d * (4 + 4 + 8) + d * (4 + 4 + 2) + 8), "flops": n * case["C"] * d * 14}
    if kind == "segments":
        bh, nk = case["B"] * case["H"], case["S"] * case["Nk"]
        pairs, rows, keys = bh * case["Nq"] * nk, bh * case["Nq"], bh * nk
        return {"bytes": rows * (d * (2 + 2 + 4 + 4) + 4) + keys * d * (2 + 2 + 4 + 4), "flops": 14 * pairs * d}
    bh, n = case["B"] * case["H"], case["N"]
    if kind == "fwd":
        return {"bytes": bh * n * (d * (6 + 4) + 4), "flops": 4 * bh * n * n * d}
    grads = 2 if kind == "train" else 4
    dout = 4 if kind == "train" else 2
    return {"bytes": bh * n * (d * (6 + dout + 4 + 3 * grads) + 4), "flops": 14 * bh * n * n * d}


def tolerance(case):
    kind = case["kind"]
    if kind == "layouts":
        return "exact"
    if kind == "channels":  # fp32 sums of bf16 inputs
        return {"rel": 2e-6, "max": 2e-3}
    # P and dS are bf16 operands of fp32 sums: about 1.7e-3 off in O, 2.4e-3 in the gradients
    return {"rel": 7e-3 if kind == "fwd" else 1e-2, "max": 0.2}


_EXACT_PAIRS = 8e10  # scores that 64-bit torch works through in a few seconds


def _exact_rows(q, k, v, do, scale, chunk):
    """(o, lse, dq, dk, dv) of one head in 64 bits; the last three are None without do."""
    q, k, v = q.double(), k.double(), v.double()
    o, lse = torch.empty((q.shape[0], v.shape[1]), dtype=torch.float64, device=q.device), []
    dq = dk = dv = None
    if do is not None:
        do, dq, dk, dv = do.double(), torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    kt, vt = k.t().contiguous(), v.t().contiguous()
    for i in range(0, q.shape[0], chunk):
        at = slice(i, i + chunk)
        s = (q[at] @ kt).mul_(scale)
        l = torch.logsumexp(s, dim=1)
        p = s.sub_(l[:, None]).exp_()
        o[at] = p @ v
        lse.append(l)
        if do is not None:
            dv += p.t() @ do[at]
            ds = (do[at] @ vt).sub_((do[at] * o[at]).sum(1, keepdim=True)).mul_(p)
            dq[at] = (ds @ k).mul_(scale)
            dk += (ds.t() @ q[at]).mul_(scale)
    return o, torch.cat(lse), dq, dk, dv


def _heads(q, k, v, do):
    B, H, N, d = q.shape
    scale, chunk = 1.0 / math.sqrt(d), max(64, min(N, (1 << 28) // max(1, k.shape[2])))
    rows = [_exact_rows(q[b, h], k[b, h], v[b, h], None if do is None else do[b, h], scale, chunk)
            for b in range(B) for h in range(H)]
    return [None if x[0] is None else torch.stack(x).reshape((B, H) + tuple(x[0].shape)) for x in zip(*rows)]


def exact(case, seed):
    kind = case["kind"]
    if kind == "layouts":
        return None
    if kind == "channels":
        if case["M"] * case["H"] * case["C"] * case["d"] > 1 << 30:
            return None
        q, k, v, do = (x.double() for x in _channels(case, seed))
        scale = 1.0 / math.sqrt(case["d"])
        s = (k * q[None, :, None, :]).sum(-1) * scale
        lse = torch.logsumexp(s, dim=-1)
        p = torch.exp(s - lse[..., None])
        o = (p[..., None] * v).sum(2)
        ds = p * ((v * do[:, :, None, :]).sum(-1) - (do * o).sum(-1)[..., None])
        dk = scale * ds[..., None] * q[None, :, None, :]
        dq = scale * (ds[..., None] * k).sum(2).sum(0)
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": p[..., None] * do[:, :, None, :]}
    if kind == "segments":
        if case["B"] * case["H"] * case["Nq"] * case["Nk"] * case["S"] > _EXACT_PAIRS:
            return None
        q, ks, vs, do = _segments(case, seed)
        o, lse, dq, dk, dv = _heads(q, torch.cat(ks, 2), torch.cat(vs, 2), do)
        return {"o": o, "lse": lse, "dq": dq, "dk": list(dk.split(case["Nk"], 2)), "dv": list(dv.split(case["Nk"], 2))}
    if case["B"] * case["H"] * case["N"] ** 2 > _EXACT_PAIRS:
        return None
    x = _qkv_do(case, seed)
    o, lse, dq, dk, dv = _heads(x[0], x[1], x[2], x[3] if len(x) > 3 else None)
    if kind == "fwd":
        return {"o": o, "lse": lse}
    if kind == "train":
        return {"o": o, "dq": dq, "dk": dk, "dv": dv}
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
