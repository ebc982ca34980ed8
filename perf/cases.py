"""The framework's work as a user runs it, as cases to be timed and compared.

A case is one pass through the public entry points (Session, HeadSession):

  step  one training step of an LSTM stack under structured dropout: masks,
        forward, MSE loss gradient, back-propagation with every gradient
  lm    one training step of a language model: masks of the stack and of the
        output site, forward, output head (FC layer, softmax cross-entropy)
        forward and backward, the stack's backward, the embedding gradient
  head  the output head alone, forward and backward
  eval  the forward pass alone without dropout (evaluation)

Sizes of the listed cases are those of the repository's workloads where it has
one.  Inputs are drawn on the GPU from the seed alone.
"""
import math
import types

import numpy as np
import torch

from paper_2106_12089_amd.session import HeadSession, Session

DEV = "cuda:0"


def _case(name, kind, L, D, I, H, B, T, dtype, p_nr, p_rh, lengths=False, V=0, p_out=0.0, x_std=0.1, w=0.0):
    """p_nr, p_rh: a rate, or a text with one rate per layer.  w: half width of
    the uniform weight distribution, 0 = 1/sqrt(H)."""
    return dict(name=name, kind=kind, layers=L, dirs=D, input=I, hidden=H, batch=B, seq=T, dtype=dtype, p_nr=p_nr,
                p_rh=p_rh, lengths=lengths, vocab=V, p_out=p_out, x_std=x_std, w=w)


def listed():
    return [
        # the smallest call: a toy stack in fp32, bound by launches and latency
        _case("tiny_f32", "step", 2, 1, 32, 64, 4, 8, "f32", 0.5, 0.5),
        # a BiLSTM sequence tagger, both directions of one layer
        _case("tagger", "step", 1, 2, 300, 256, 32, 40, "bf16", 0.5, 0.5, x_std=1.0),
        # the medium language model's LSTM stack, non-recurrent dropout: the headline step
        _case("lm_medium", "step", 2, 1, 650, 650, 20, 35, "bf16", 0.5, 0.0, x_std=0.05, w=0.05),
        # the same stack in fp32 with recurrent dropout too (a user who checks in full precision)
        _case("lm_medium_f32", "step", 2, 1, 650, 650, 20, 35, "f32", 0.5, 0.5, x_std=0.05, w=0.05),
        # the whole training step of that language model, with its vocabulary
        _case("lm_medium_train", "lm", 2, 1, 650, 650, 20, 35, "bf16", 0.5, 0.5, V=10000, p_out=0.5, x_std=0.05,
              w=0.05),
        # its evaluation: the forward pass without dropout
        _case("lm_medium_eval", "eval", 2, 1, 650, 650, 20, 35, "bf16", 0.0, 0.0, x_std=0.05, w=0.05),
        # the large language model's stack (wide recurrence, small batch)
        _case("lm_large", "step", 2, 1, 1500, 1500, 20, 35, "bf16", 0.65, 0.65, x_std=0.04, w=0.04),
        # three layers with a dropout rate for each layer and site, long sequence
        _case("awd_lstm", "step", 3, 1, 400, 1150, 20, 70, "bf16", "0.4,0.25,0.25", "0.5,0.5,0.5"),
        # a translation encoder: padded sentences of different lengths
        _case("seq2seq_enc", "step", 2, 1, 500, 500, 64, 50, "bf16", 0.3, 0.0, lengths=True),
        # the translation model's output projection, sized by the vocabulary
        _case("seq2seq_head", "head", 2, 1, 500, 500, 64, 50, "bf16", 0.0, 0.0, lengths=True, V=20000, p_out=0.3),
        # a bidirectional stack at sizes that fit no tile, batch between the small and the large paths
        _case("ragged_bi", "step", 2, 2, 203, 211, 37, 29, "bf16", 0.3, 0.5, lengths=True, x_std=0.5),
        # a large batch: every product is a large matrix product
        _case("large_batch", "step", 2, 1, 1024, 1024, 256, 64, "bf16", 0.5, 0.5, x_std=1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "lm", "head", "eval"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    while True:
        L, D = rng.choice([1, 2, 2, 3]), rng.choice([1, 1, 1, 2])
        I, H = _log_int(rng, 32, 1500), _log_int(rng, 40, 1500)
        B, T = _log_int(rng, 1, 256), _log_int(rng, 4, 70)
        if dtype == "f32" and (H > 650 or B > 64) or H > 1024 and B > 64:
            continue
        if kind == "lm" and B > 64:
            continue
        # a third of the largest listed step at most
        if D * H <= 1024 and L * D * T * B * H * (I + H) <= 2 * 64 * 256 * 1024 * 2048 / 3:
            break
        if D == 1 and L * T * B * H * (I + H) <= 2 * 64 * 256 * 1024 * 2048 / 3:
            break
    V = 0
    if kind in ("lm", "head"):
        V = 4 * _log_int(rng, 250, 5000)
        T = max(2, min(T, int(2.5e7 / (B * V))))
    p_nr, p_rh = rng.choice([0.3, 0.5, 0.65]), rng.choice([0.0, 0.3, 0.5])
    if kind == "eval":
        p_nr = p_rh = 0.0
    return dict(kind=kind, layers=L, dirs=D, input=I, hidden=H, batch=B, seq=T, dtype=dtype, p_nr=p_nr, p_rh=p_rh,
                lengths=kind != "eval" and rng.random() < 0.4, vocab=V, p_out=rng.choice([0.3, 0.5]) if V else 0.0,
                x_std=rng.choice([0.05, 0.2, 1.0]), w=0.0)


def _rates(p, L):
    return [float(v) for v in p.split(",")] if isinstance(p, str) else [float(p)] * L


def _kin(c, l):
    return c["input"] if l == 0 else c["dirs"] * c["hidden"]


def _inputs(c, seed):
    """Seeded inputs on the GPU, values as the path takes them (bf16 where it
    stores bf16), float32."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + 17)
    L, D, I, H, B, T, V = (c[k] for k in ("layers", "dirs", "input", "hidden", "batch", "seq", "vocab"))
    q = (lambda a: a.to(torch.bfloat16).float()) if c["dtype"] == "bf16" else (lambda a: a)
    uni = lambda *s: (torch.rand(*s, generator=g, device=DEV) * 2 - 1) * (c["w"] or 1 / math.sqrt(H))
    nor = lambda *s: torch.randn(*s, generator=g, device=DEV)
    n = types.SimpleNamespace()
    n.lengths = None
    if c["lengths"]:
        n.lengths = torch.randint(max(1, (2 * T) // 5), T + 1, (B,), generator=g, device=DEV)
    if c["kind"] != "head":
        n.W = [q(uni(_kin(c, l), 4 * H)) for l in range(L) for _ in range(D)]
        n.U = [q(uni(H, 4 * H)) for _ in range(L * D)]
        n.b = [uni(4 * H) for _ in range(L * D)]
        n.h0, n.c0 = q(0.1 * nor(L * D, B, H)), 0.1 * nor(L * D, B, H)
        n.target = nor(T, B, D * H)
    if V:
        zipf = torch.arange(1, V + 1, device=DEV, dtype=torch.float32) ** -1.1
        n.tokens = torch.multinomial(zipf, T * B, replacement=True, generator=g).reshape(T, B)
        n.targets = torch.multinomial(zipf, T * B, replacement=True, generator=g).reshape(T, B)
        n.W_fc, n.b_fc = q(uni(D * H, V)), uni(V)
    if c["kind"] == "lm":
        n.x = (c["x_std"] * nor(V, I))[n.tokens]
    elif c["kind"] == "head":
        n.y = torch.tanh(0.5 * nor(T, B, D * H))         # a top LSTM output
    else:
        n.x = c["x_std"] * nor(T, B, I)
    if c["kind"] != "head":
        if n.lengths is not None:                          # padded positions carry zero input
            n.x = n.x * (torch.arange(T, device=DEV)[:, None] < n.lengths[None, :])[:, :, None]
        n.x = q(n.x)
    return n


def prepare(case, seed):
    c, n = case, _inputs(case, seed)
    h = lambda v: v.cpu().numpy() if isinstance(v, torch.Tensor) else [t.cpu().numpy() for t in v] if v else v
    wl = types.SimpleNamespace(**{k: h(v) for k, v in vars(n).items() if k != "y"})
    wl.cfg = types.SimpleNamespace(num_layers=c["layers"], num_dirs=c["dirs"], hidden=c["hidden"], dtype=c["dtype"],
                                   loss="mse")
    s = types.SimpleNamespace(case=c, seed=int(seed), lstm=None, head=None)
    if c["kind"] != "head":
        s.lstm = Session(wl, _rates(c["p_nr"], c["layers"]), _rates(c["p_rh"], c["layers"]), 1, DEV)
    else:
        wl.x = np.zeros((c["seq"], c["batch"], 1), np.float32)
        s.y = n.y
    if c["vocab"]:
        s.head = HeadSession(wl, c["p_out"], 1, DEV)
    if c["kind"] == "lm":
        s.tokens = n.tokens.to(torch.int32).contiguous()
        s.d_emb = torch.zeros(c["vocab"], c["input"], device=DEV)
    if c["kind"] == "eval":
        s.lstm.masks(s.seed, 0)                            # no dropout: the same lists for every call
    return s


def run(s):
    kind, m, hd = s.case["kind"], s.lstm, s.head
    if kind == "eval":
        m.forward()
        return {"y": m.y, "hT": m.hT, "cT": m.cT}
    out = {}
    if kind == "step":
        m.step(s.seed, 1)
        out["loss"] = m.loss
    else:
        hd.masks(s.seed, 1)
        if kind == "lm":
            m.masks(s.seed, 1)
            m.forward()
        hd.forward(m.y if kind == "lm" else s.y)
        hd.backward()
        out.update(logits=hd.logits, loss=hd.loss, dy=hd.dy, dW_fc=hd.dW, db_fc=hd.db)
        if kind == "lm":
            m.backward(dy=hd.dy)
            s.d_emb.zero_()
            m.embedding_backward(s.tokens, s.case["vocab"], s.d_emb)
            out["d_emb"] = s.d_emb
    if m is not None:
        out.update(y=m.y, hT=m.hT, cT=m.cT, dx=m.dx, dh0=m.dh0, dc0=m.dc0, dW=m.dW, dU=m.dU, db=m.db)
    return out


def work(case):
    c = case
    L, D, I, H, B, T, V = (c[k] for k in ("layers", "dirs", "input", "hidden", "batch", "seq", "vocab"))
    es, G, F = (2 if c["dtype"] == "bf16" else 4), 4 * H, D * H
    flops = byt = 0.0
    train = c["kind"] in ("step", "lm")
    if c["kind"] != "head":
        pn, pr = _rates(c["p_nr"], L), _rates(c["p_rh"], L)
        mac = sum(D * T * B * G * ((1 - pn[l]) * _kin(c, l) + (1 - pr[l]) * H) for l in range(L))
        par = sum(D * G * (_kin(c, l) + H) for l in range(L))
        st = L * D * B * H
        flops += 2 * mac * (3 if train else 1)            # kept rows only, forward and both gradients
        byt += T * B * I * es + par * es + L * D * G * 4 + st * (es + 4) + T * B * F * 4 + 2 * st * 4
        if train:
            byt += T * B * I * 4 + 2 * st * 4 + par * 4 + L * D * G * 4
        if c["kind"] == "step":
            byt += T * B * F * 4                           # the target
    if V:
        flops += 3 * 2.0 * T * B * F * (1 - c["p_out"]) * V
        byt += F * V * (es + 4) + 2 * V * 4 + T * B * V * 4 + 2 * T * B * F * 4 + 2 * T * B * 4
        if c["kind"] == "lm":
            byt += min(V, T * B) * I * 4
    return {"bytes": byt, "flops": flops}


def tolerance(case):
    """About four times the error of these paths against 64 bits: at most
    1.7e-6 (fp32) and 3e-3 (bf16: rounded copies of h, da and dz) in any output
    of the listed and of drawn cases."""
    return {"rel": 8e-6} if case["dtype"] == "f32" else {"rel": 1e-2}


# -- the same results in 64 bits, in plain torch ------------------------------
def _keep(seed, step, sid, T, K, p):
    """Keep bits [T][K]: neuron k is dropped at t iff word k%4 of Philox4x64-10
    at counter (k/4, t, sid, step), key (seed, 0), is below floor(p 2^64)."""
    m = np.ones((T, K), np.bool_)
    thr = int(p * 2 ** 64) if p > 0 else 0
    for t in range(T if p > 0 else 0):
        c = ((t << 64) + (sid << 128) + (step << 192) - 1) % 2 ** 256    # numpy's generator counts up first
        words = np.random.Philox(counter=c, key=seed).random_raw((K + 3) // 4 * 4)
        m[t] = words[:K] >= np.uint64(thr)
    return torch.from_numpy(m).to(DEV).double() / (1.0 - p)


def exact(case, seed):
    c, n = case, _inputs(case, seed)
    L, D, H, B, T, V = (c[k] for k in ("layers", "dirs", "hidden", "batch", "seq", "vocab"))
    kind, F, train = c["kind"], D * H, c["kind"] in ("step", "lm")
    dbl = lambda t: t.double().requires_grad_(True)
    valid = torch.ones(T, B, dtype=torch.bool, device=DEV)
    if n.lengths is not None:
        valid = torch.arange(T, device=DEV)[:, None] < n.lengths[None, :]
    out = {}
    if kind != "head":
        pn, pr = _rates(c["p_nr"], L), _rates(c["p_rh"], L)
        W, U, b = [dbl(t) for t in n.W], [dbl(t) for t in n.U], [dbl(t) for t in n.b]
        x, h0, c0 = dbl(n.x), dbl(n.h0), dbl(n.c0)
        cur, hT, cT = x, [], []
        with torch.set_grad_enabled(train):
            for l in range(L):
                xm = cur * _keep(int(seed), 1, 4 * l, T, _kin(c, l), pn[l])[:, None, :]
                halves = []
                for d in range(D):
                    k = l * D + d
                    mr = _keep(int(seed), 1, 4 * l + 2 + d, T, H, pr[l])
                    gx = xm @ W[k] + b[k]
                    h, cc, ys = h0[k], c0[k], [None] * T
                    for t in (range(T) if d == 0 else range(T - 1, -1, -1)):
                        a = gx[t] + (h * mr[t]) @ U[k]
                        i, f, gg, o = a[:, :H], a[:, H:2 * H], a[:, 2 * H:3 * H], a[:, 3 * H:]
                        cn = torch.sigmoid(f) * cc + torch.sigmoid(i) * torch.tanh(gg)
                        hn = torch.sigmoid(o) * torch.tanh(cn)
                        v = valid[t][:, None]
                        h, cc = torch.where(v, hn, h), torch.where(v, cn, cc)
                        ys[t] = torch.where(v, hn, torch.zeros_like(hn))
                    hT.append(h)
                    cT.append(cc)
                    halves.append(torch.stack(ys))
                cur = torch.cat(halves, 2)
        y = cur
        out.update(y=y.detach(), hT=torch.stack(hT).detach(), cT=torch.stack(cT).detach())
        if kind == "eval":
            return out
    else:
        y = dbl(n.y)
    if V:
        Wf, bf = dbl(n.W_fc), dbl(n.b_fc)
        yl = y.detach().requires_grad_(True)
        z = (yl * _keep(int(seed), 1, 4 * L, T, F, c["p_out"])[:, None, :]) @ Wf + bf
        nll = torch.logsumexp(z, 2) - torch.gather(z, 2, n.targets[:, :, None])[:, :, 0]
        loss = (nll * valid).sum() / valid.sum()
        dy, dWf, dbf = torch.autograd.grad(loss, [yl, Wf, bf])
        out.update(logits=z.detach(), loss=loss.detach().reshape(1), dy=dy, dW_fc=dWf, db_fc=dbf)
        if kind == "head":
            return out
    else:
        dif = (y - n.target.double()) * valid[:, :, None]
        loss = (dif.detach() ** 2).sum() / (valid.sum() * F)
        dy = 2 * dif.detach() / (valid.sum() * F)
        out["loss"] = loss.reshape(1)
    g = torch.autograd.grad(y, [x, h0, c0, *W, *U, *b], dy)
    k = L * D
    out.update(dx=g[0], dh0=g[1], dc0=g[2], dW=list(g[3:3 + k]), dU=list(g[3 + k:3 + 2 * k]), db=list(g[3 + 2 * k:]))
    if kind == "lm":
        e = torch.zeros(V, c["input"], dtype=torch.float64, device=DEV)
        out["d_emb"] = e.index_add_(0, n.tokens.reshape(-1), g[0].reshape(T * B, -1))
    return out
