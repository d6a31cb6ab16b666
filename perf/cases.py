"""The work that a program using this framework has it do, as cases that can be timed.

Three kinds of program call the public entry points:

* a serving loop drafts with the chain of heads once per denoising step (``MrpContext.chain_step`` with the MLP
  head body, ``chain_step_tf`` with the transformer body), commits what was revealed (``commit``) and, when it
  decodes speculatively, checks the drafts against the backbone's logits (``verify_accept``,
  ``verify_accept_joint``);
* a training loop takes the head's objective and its gradient (``kl_loss``);
* an analysis script reduces recorded block states to residual magnitudes (``residual_rms``).

The sizes are those of the benchmark configurations and of the tests, and generic ones between them: one
sequence or hundreds, blocks of 4 to 16 positions, hidden sizes 256 to 4096, vocabularies of 4096 to 151936
entries, some of them odd.

Inputs are drawn on the GPU from the seed: weights N(0, 0.02), hidden states N(0, 1), logits N(0, 2) with one
peaked entry per row (8 to 20 above the rest, as a language model's rows have one likely token, more or less
certain), caches N(0, 1) with prefix lengths over the whole range.
"""
from __future__ import annotations

import math

import torch

import paper_2605_18817_amd as mrp


def listed():
    return [
        # one sequence of the smallest configuration: a chain of short launches, where latency is all
        dict(name="chain_tiny", kind="chain", d=256, V=4096, B=1, L=4, K=3, tau=0.9, tau_remask=-1.0, commit=False),
        # one interactive user drafting with the small backbone's sizes: four rows against the whole LM head
        dict(name="chain_one_sequence", kind="chain", d=2048, V=151936, B=1, L=4, K=3, tau=0.9, tau_remask=-1.0, commit=False),
        # a served batch at those sizes (128 rows), the configuration that the drafting rate is quoted on
        dict(name="chain_draft", kind="chain", d=2048, V=151936, B=32, L=4, K=3, tau=0.9, tau_remask=-1.0, commit=False),
        # a vocabulary that is not a multiple of 4, at the row count of a dozen sequences
        dict(name="chain_odd_vocab", kind="chain", d=2048, V=50257, B=12, L=16, K=3, tau=0.9, tau_remask=-1.0, commit=True),
        # the large backbone's sizes with a ragged batch (592 rows)
        dict(name="chain_ragged_batch", kind="chain", d=4096, V=151936, B=37, L=16, K=3, tau=0.9, tau_remask=-1.0, commit=True),
        # ... with the batch of its drafting configuration (1024 rows)
        dict(name="chain_block", kind="chain", d=4096, V=151936, B=64, L=16, K=3, tau=0.9, tau_remask=-1.0, commit=False),
        # ... and the largest configuration: low threshold with remasking, 4096 rows, committed at the end of the step
        dict(name="chain_remask", kind="chain", d=4096, V=151936, B=256, L=16, K=3, tau=0.5, tau_remask=0.3, commit=True),
        # transformer head body (three layers, one module applied three times) at the small backbone's sizes
        dict(name="tf_draft", kind="tf", d=2048, V=151936, B=32, L=4, K=3, D=3, nh=16, nkv=8, ff=6144, P=1024, tau=0.9),
        # ... and at the large backbone's, 24 sequences of 16 positions
        dict(name="tf_block", kind="tf", d=4096, V=151936, B=24, L=16, K=3, D=3, nh=32, nkv=8, ff=12288, P=1024, tau=0.9),
        # speculative verification of three drafts for each of 128 sequences
        dict(name="verify", kind="verify", V=151936, B=128, L=16, K=3, joint=False),
        # the training objective of 1024 rows with its gradient
        dict(name="kl_training", kind="kl", V=151936, M=1024, grad=True, share=1.0),
        # residual magnitudes of eight recorded blocks of 16 positions (17 states each) of logits
        dict(name="residual_logits", kind="rms", n=8, S=17, N=16 * 151936, bf16=False),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _vocab(rng):
    return rng.choice([151936, 151936, 151936, 32000, 50257, _log(rng, 4096, 151936)])


def draw(rng):
    """One more case of the same ranges; none costs more than chain_remask."""
    kind = rng.choice(["chain"] * 6 + ["tf"] * 3 + ["verify", "kl", "rms"])
    L = rng.choice([4, 8, 16])
    if kind == "chain":
        d = rng.choice([256, 1024, 2048, 2048, 2560, 4096, 4096, 4096])
        remask = rng.random() < 0.4
        return dict(kind=kind, d=d, V=_vocab(rng), B=_log(rng, 1, 4096 // L), L=L, K=rng.choice([1, 2, 3]),
                    tau=rng.choice([0.5, 0.9]), tau_remask=0.3 if remask else -1.0, commit=rng.random() < 0.5)
    if kind == "tf":
        d, nh, nkv, ff, top = rng.choice([(1024, 8, 4, 3072, 1024), (2048, 16, 8, 6144, 1024), (4096, 32, 8, 12288, 512)])
        return dict(kind=kind, d=d, V=_vocab(rng), B=_log(rng, 1, top // L), L=L, K=rng.choice([1, 2, 3]),
                    D=rng.choice([1, 2, 3]), nh=nh, nkv=nkv, ff=ff, P=rng.choice([128, 512, 1024]), tau=0.9)
    if kind == "verify":
        K, joint = rng.choice([1, 2, 3, 4]), rng.random() < 0.5
        return dict(kind=kind, V=_vocab(rng), B=_log(rng, 1, 128 // (2 if joint else 1)), L=L, K=K, joint=joint)
    if kind == "kl":
        return dict(kind=kind, V=_vocab(rng), M=_log(rng, 16, 2048), grad=rng.random() < 0.6, share=rng.choice([0.5, 1.0]))
    S, bf16 = rng.choice([5, 9, 17]), rng.random() < 0.5
    N = (S - 1) * rng.choice([1024, 2048, 4096, 50257, 151936])
    most = max(1, int(1.3e9 / (S * N * (2 if bf16 else 4))))
    return dict(kind=kind, n=_log(rng, 1, min(400, most)), S=S, N=N, bf16=bf16)


# ---- what a program holds before the call ------------------------------------------------------------------


def _normal(g, *shape, std=1.0, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)


def _body(g, rows, cols):
    """A head-body weight in the form that the library takes."""
    return mrp.pack_weight(_normal(g, rows, cols, std=0.02), body=True)


def _logits(g, M, V):
    z = _normal(g, M, V, std=2.0, dtype=torch.float32)
    peak = torch.randint(V, (M, 1), device="cuda", generator=g)
    z.scatter_add_(1, peak, torch.empty(M, 1, device="cuda").uniform_(8.0, 20.0, generator=g))
    return z


def _ones(n):
    return torch.ones(n, dtype=torch.bfloat16, device="cuda")


def prepare(case, seed):
    c, g = dict(case), torch.Generator(device="cuda")
    g.manual_seed(seed)
    s = {"c": c}
    if c["kind"] in ("chain", "tf"):
        d, V, B, L, K = c["d"], c["V"], c["B"], c["L"], c["K"]
        M = B * L
        s["ctx"] = mrp.MrpContext(d, V, M, L)
        s["E"] = _normal(g, V, d, std=0.02)
        s["W"] = mrp.pack_weight(_normal(g, V, d, std=0.02))
        s["h"] = _normal(g, M, d)
        s["z"] = _logits(g, M, V)
        s["h_run"] = torch.zeros(M, d, dtype=torch.float32, device="cuda")
        s["io"] = mrp.StepIO(B, L, K)
        s["cfg"] = mrp.RevealCfg(tau=c["tau"], tau_remask=c.get("tau_remask", -1.0), fresh_block=1)
        if c["kind"] == "chain":
            s["heads"] = [mrp.Head(_body(g, d, 2 * d), _body(g, d, d), _ones(d)) for _ in range(K)]
            s["x_out"] = torch.full((M,), -1, dtype=torch.int32, device="cuda")
            s["n_masked"] = torch.zeros(B, dtype=torch.int32, device="cuda")
        else:
            D, nh, nkv, ff, P = c["D"], c["nh"], c["nkv"], c["ff"], c["P"]
            s["ctx"].tbody_create(D, nh, nkv, ff, P)
            s["heads"] = [mrp.Head(_body(g, d, 2 * d), None, _ones(d))] * K
            s["layers"] = [mrp.TLayer(_body(g, (nh + 2 * nkv) * 128, d), _body(g, d, nh * 128), _body(g, 2 * ff, d),
                                      _body(g, d, ff), _ones(d), _ones(d), _normal(g, B, P, nkv, 128),
                                      _normal(g, B, P, nkv, 128)) for _ in range(D)] * K
            plen = torch.randint(P + 1, (B,), device="cuda", generator=g, dtype=torch.int32)
            plen[0], plen[-1] = 0, P
            s["prefix_len"] = plen
    elif c["kind"] == "verify":
        V, B, L, K = c["V"], c["B"], c["L"], c["K"]
        J = K + 1 if c["joint"] else 1
        s["ctx"] = mrp.MrpContext(128, V, B * L, L)
        v = _normal(g, B, J, L, V, std=2.0, dtype=torch.float32)
        pos = torch.argsort(torch.rand(B, L, device="cuda", generator=g), dim=1)[:, :K]
        tok = torch.randint(V, (B, K), device="cuda", generator=g)
        hit = torch.rand(B, K, device="cuda", generator=g) < 0.7     # the backbone agrees with most drafts
        b = torch.arange(B, device="cuda").unsqueeze(1).expand(B, K)
        j = torch.arange(K, device="cuda").expand(B, K) if c["joint"] else torch.zeros_like(b)
        v[b, j, pos, tok] += 12.0 * hit
        s["verify"], s["pos"], s["tok"] = v, pos.int().contiguous(), tok.int().contiguous()
        s["match"] = torch.zeros(B, K, dtype=torch.uint8, device="cuda")
        s["len"] = torch.zeros(B, dtype=torch.int32, device="cuda")
        s["fix"] = torch.zeros(B, dtype=torch.int32, device="cuda")
    elif c["kind"] == "kl":
        V, M = c["V"], c["M"]
        s["ctx"] = mrp.MrpContext(128, V, M, 1)
        s["teacher"] = _logits(g, M, V)
        s["student"] = s["teacher"] + _normal(g, M, V, std=0.5, dtype=torch.float32)
        s["mask"] = None if c["share"] >= 1 else (torch.rand(M, device="cuda", generator=g) < c["share"]).to(torch.uint8)
        s["loss"] = torch.zeros(M, dtype=torch.float32, device="cuda")
        s["grad"] = torch.zeros(M, V, dtype=torch.float32, device="cuda") if c["grad"] else None
    else:
        n, S, N = c["n"], c["S"], c["N"]
        s["ctx"] = mrp.MrpContext(128, 1024, 16, 16)
        x = torch.empty(n, S, N, dtype=torch.bfloat16 if c["bf16"] else torch.float32, device="cuda")
        for i in range(n):      # a walk: the first state N(0, 2), every further one N(0, 0.4) away from the one before
            w = _normal(g, S, N, std=0.4, dtype=torch.float32)
            w[0] *= 5.0
            x[i] = torch.cumsum(w, 0)
        s["X"] = x
        s["pair"] = torch.zeros(n, S, S, dtype=torch.float64, device="cuda")
        s["delta"] = torch.zeros(S, dtype=torch.float64, device="cuda")
    return s


# ---- one pass ----------------------------------------------------------------------------------------------


def run(s):
    c, ctx = s["c"], s["ctx"]
    if c["kind"] in ("chain", "tf"):
        io = s["io"]
        if c["kind"] == "chain":
            ctx.chain_step(c["B"], c["K"], s["h"], s["h_run"], s["E"], s["W"], s["heads"], s["z"], s["cfg"], io)
        else:
            ctx.chain_step_tf(c["B"], c["K"], s["h"], s["h_run"], s["E"], s["W"], s["heads"], s["layers"],
                              s["prefix_len"], s["z"], s["cfg"], io)
        out = dict(z=s["z"], h_run=s["h_run"], tok=io.tok, conf=io.conf, lse=io.lse, masked=io.masked,
                   revealed_at=io.revealed_at, cond_tok=io.cond_tok, draft_pos=io.draft_pos, draft_tok=io.draft_tok,
                   remasked=io.remasked, x_tok=io.x_tok)
        if c.get("commit"):
            ctx.commit(c["B"], io.x_tok, io.revealed_at, io.masked, s["x_out"], s["n_masked"])
            out.update(x_out=s["x_out"], n_masked=s["n_masked"])
        return out
    if c["kind"] == "verify":
        call = ctx.verify_accept_joint if c["joint"] else ctx.verify_accept
        call(c["B"], c["K"], s["verify"], s["pos"], s["tok"], c["K"], s["match"], s["len"], s["fix"])
        return dict(match=s["match"], accept_len=s["len"], correction_tok=s["fix"])
    if c["kind"] == "kl":
        ctx.kl_loss(c["M"], s["teacher"], s["student"], s["mask"], 1.0 / c["M"], s["loss"], s["grad"])
        return dict(loss=s["loss"], grad=s["grad"]) if c["grad"] else dict(loss=s["loss"])
    ctx.residual_rms(c["n"], c["S"], c["N"], s["X"], c["bf16"], s["pair"], s["delta"])
    return dict(pair=s["pair"], delta=s["delta"])


# ---- the same pass in 64 bits ---------------------------------------------------------------------------------


def _matmul(x, w):
    """x w^T in 64 bits, a slice of the weight's rows at a time."""
    return torch.cat([x @ r.double().t() for r in w.split(32768)], dim=1)


def _norm64(u):
    return u * torch.rsqrt(u.pow(2).mean(1, keepdim=True) + 1e-6)


def _layer64(c, u, layer, plen):
    """One decoder layer of the transformer body on u [M][d]."""
    (wqkv, wo, wgu, wdown, kc, vc), B, L, P, nh, nkv = layer, c["B"], c["L"], c["P"], c["nh"], c["nkv"]
    qkv = _matmul(_norm64(u), wqkv).view(B, L, nh + 2 * nkv, 128)
    pos = plen.double().view(B, 1) + torch.arange(L, device="cuda", dtype=torch.float64)
    ang = (pos.unsqueeze(2) * 1.0e6 ** (-torch.arange(64, device="cuda", dtype=torch.float64) / 64)).unsqueeze(2)
    x0, x1 = qkv[..., :64], qkv[..., 64:]
    rot = torch.cat([x0 * ang.cos() - x1 * ang.sin(), x1 * ang.cos() + x0 * ang.sin()], dim=3)
    q, k, v = rot[:, :, :nh], rot[:, :, nh:nh + nkv], qkv[:, :, nh + nkv:]
    seen = torch.cat([torch.arange(P, device="cuda") < plen.view(B, 1), torch.ones(B, L, dtype=torch.bool, device="cuda")], 1)
    keys = torch.cat([kc.double(), k], 1).permute(0, 2, 1, 3).contiguous()
    vals = torch.cat([vc.double(), v], 1).permute(0, 2, 1, 3).contiguous()
    q = q.reshape(B, L, nkv, nh // nkv, 128).permute(0, 2, 3, 1, 4).reshape(B, nkv, -1, 128)
    w = (q @ keys.transpose(2, 3).contiguous()) / math.sqrt(128.0)
    w = torch.softmax(w.masked_fill(~seen.view(B, 1, 1, -1), -math.inf), -1)
    o = (w @ vals).view(B, nkv, nh // nkv, L, 128).permute(0, 3, 1, 2, 4).reshape(B * L, nh * 128)
    a = u + _matmul(o, wo)
    gate, up = _matmul(_norm64(a), wgu).chunk(2, dim=1)
    return a + _matmul(gate * torch.sigmoid(gate) * up, wdown)


def _chain64(c, g):
    d, V, B, L, K = c["d"], c["V"], c["B"], c["L"], c["K"]
    M, tau, tau_r = B * L, c["tau"], c.get("tau_remask", -1.0)
    E, W = _normal(g, V, d, std=0.02), _normal(g, V, d, std=0.02)
    h, z = _normal(g, M, d).double(), _logits(g, M, V)
    if c["kind"] == "chain":
        heads = [(_normal(g, d, 2 * d, std=0.02), _normal(g, d, d, std=0.02)) for _ in range(K)]
    else:
        w1 = _normal(g, d, 2 * d, std=0.02)
        o = c["nh"] * 128
        layers = [tuple(_normal(g, r, k, std=0.02) for r, k in (((c["nh"] + 2 * c["nkv"]) * 128, d), (d, o), (2 * c["ff"], d), (d, c["ff"])))
                  + (_normal(g, B, c["P"], c["nkv"], 128), _normal(g, B, c["P"], c["nkv"], 128)) for _ in range(c["D"])]
        plen = torch.randint(c["P"] + 1, (B,), device="cuda", generator=g, dtype=torch.int32)
        plen[0], plen[-1] = 0, c["P"]
    z = z.double()
    rows = torch.arange(B, device="cuda")
    masked = torch.ones(B, L, dtype=torch.bool, device="cuda")
    at = torch.full((B, L), -1, device="cuda")
    cond, prot, confs, lses = None, None, [], []
    for k in range(K + 1):
        if k:
            x = torch.cat([h, E[cond].double().repeat_interleave(L, 0)], 1)
            if c["kind"] == "chain":
                a = _matmul(x, heads[k - 1][0])
                u = _matmul(a * torch.sigmoid(a), heads[k - 1][1])
            else:
                u = _matmul(x, w1)
                for layer in layers:
                    u = _layer64(c, u, layer, plen)
            h = h + u
            z += _matmul(_norm64(u).bfloat16().double(), W)      # the LM head takes its operand in bf16
        lse = torch.logsumexp(z, 1)
        top, tok = z.max(1)
        conf, tok = torch.exp(top - lse).view(B, L), tok.view(B, L)
        confs.append(conf.reshape(M))
        lses.append(lse)
        left, best = masked.any(1), torch.where(masked, conf, -1.0).argmax(1)
        new = masked & (conf > tau)
        new[rows, best] |= left                    # at least one reveal for each sequence with a masked row
        cond = tok[rows, best] if k == 0 else torch.where(left, tok[rows, best], cond)
        prot = best if k == 0 else prot
        masked, at = masked & ~new, torch.where(new, k, at)
        if k and tau_r >= 0:
            again = (at >= 0) & (at < k) & (torch.arange(L, device="cuda") != prot.unsqueeze(1)) & (conf < tau_r)
            masked, at = masked | again, torch.where(again, -1, at)
    return dict(z=z, h_run=h, conf=torch.stack(confs), lse=torch.stack(lses))


def exact(case, seed):
    """The computed numbers of one pass; None for the decisions (tokens, positions, flags)."""
    c, g = dict(case), torch.Generator(device="cuda")
    g.manual_seed(seed)
    if c["kind"] in ("chain", "tf"):
        out = _chain64(c, g)
        none = ["tok", "masked", "revealed_at", "cond_tok", "draft_pos", "draft_tok", "remasked", "x_tok"]
        return dict(out, **{n: None for n in none + (["x_out", "n_masked"] if c.get("commit") else [])})
    if c["kind"] == "kl":
        V, M = c["V"], c["M"]
        t = _logits(g, M, V)
        s = (t + _normal(g, M, V, std=0.5, dtype=torch.float32)).double()
        t = t.double()
        on = torch.ones(M, 1, device="cuda") if c["share"] >= 1 else (torch.rand(M, device="cuda", generator=g) < c["share"]).view(M, 1)
        p, q = torch.log_softmax(t, 1), torch.log_softmax(s, 1)
        out = dict(loss=((p.exp() * (p - q)).sum(1, keepdim=True) * on / M).view(M))
        return dict(out, grad=(q.exp() - p.exp()) * on / M) if c["grad"] else out
    if c["kind"] == "rms":
        n, S, N = c["n"], c["S"], c["N"]
        pair = torch.zeros(n, S, S, dtype=torch.float64, device="cuda")
        for i in range(n):
            w = _normal(g, S, N, std=0.4, dtype=torch.float32)
            w[0] *= 5.0
            x = torch.cumsum(w, 0).to(torch.bfloat16 if c["bf16"] else torch.float32).double()
            for t in range(S):
                pair[i, t, t] = x[t].pow(2).mean().sqrt()
                pair[i, t, t + 1:] = (x[t + 1:] - x[t]).pow(2).mean(1).sqrt()
        delta = [pair[:, torch.arange(1, S), torch.arange(1, S)].mean()]
        delta += [torch.diagonal(pair, r, 1, 2).mean() for r in range(1, S)]
        return dict(pair=pair, delta=torch.stack(delta))
    return None


# ---- what a pass cannot do without, and how close another correct one comes -----------------------------------


def work(case):
    c = case
    if c["kind"] in ("chain", "tf"):
        d, V, K, M = c["d"], c["V"], c["K"], c["B"] * c["L"]
        # the LM head and the logit state once each (the state read and written), the heads' weights, h in, h_run out
        nbytes = 2.0 * V * d + 8.0 * M * V + 6.0 * M * d
        flops = 2.0 * K * M * V * d
        if c["kind"] == "chain":
            nbytes += 6.0 * K * d * d
            flops += 6.0 * K * M * d * d
        else:
            qkv, o = (c["nh"] + 2 * c["nkv"]) * 128, c["nh"] * 128
            layer = d * (qkv + o + 3 * c["ff"])                       # projection weights of a layer
            pairs = c["B"] * (c["P"] / 2 + c["L"]) * c["L"] * o       # scores and values, prefixes half full on average
            nbytes += 4.0 * d * d + c["D"] * (2.0 * layer + 4.0 * c["B"] * (c["P"] / 2) * c["nkv"] * 128)
            flops += K * (4.0 * M * d * d + c["D"] * (2.0 * M * layer + 4.0 * pairs))
        return {"bytes": nbytes, "flops": flops}
    if c["kind"] == "verify":
        n = float(c["B"]) * c["K"] * c["V"]
        return {"bytes": 4.0 * n, "flops": n}
    if c["kind"] == "kl":
        n = float(c["M"]) * c["V"] * c["share"]
        return {"bytes": 8.0 * n + (4.0 * c["M"] * c["V"] if c["grad"] else 0.0), "flops": (14.0 if c["grad"] else 8.0) * n}
    n = float(c["n"]) * c["N"]
    return {"bytes": (2.0 if c["bf16"] else 4.0) * c["S"] * n, "flops": (1.5 * c["S"] * (c["S"] + 1)) * n}


def tolerance(case):
    # Each about four times what the same rows show in a smaller batch, where other kernels sum in another order.
    if case["kind"] == "chain":
        # The LM-head operand is bf16: an fp32 sum in another order moves some of its roundings (logits 5e-5 apart,
        # the farthest 8e-4), and with them one in a thousand argmaxes of rows without a clear winner.
        return {"rel": 2.5e-4, "max": 4e-3, "differ": 5e-3}
    if case["kind"] == "tf":
        return {"rel": 6e-4, "max": 6e-3, "differ": 5e-3}     # the same through three more layers: 1.5e-4 and 1.6e-3
    if case["kind"] == "verify":
        return "exact"
    if case["kind"] == "kl":
        # against 64 bits: loss 7.5e-6; gradient (a difference of two probabilities) 8.5e-6, its farthest entry 6e-3
        return {"rel": 4e-5, "max": 2.5e-2}
    return {"rel": 1e-11}                     # fp64 sums
