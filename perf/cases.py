"""The work whose speed is measured: matrix-vector products of Llama-style decode.

A program that decodes with this library calls it in four ways: one matrix at a
time (``tvl_gemv``), one item with its RMSNorm, SwiGLU pair or several x vectors
(``tvl_gemv_item``), and a plan over the matrices of one step of a layer, of a
whole layer or of a whole token (``tvl_sweep_plan_create`` once, ``run`` per
token).  The cases cover each of them, every weight type (fp32, fp16, 8- and
4-bit block-quantised), the fused options, and from a 2 MB matrix to a token of
several GB.  Weights are N(0, 0.02^2), activations N(0, 1), RMSNorm weights near
1; quantised weights come from quantising such a draw, one absolute-maximum
scale per 64 columns.
"""
from __future__ import annotations

import math

import torch

from paper_2601_03324_amd import tvl

DT = {"f32": tvl.TVL_F32, "f16": tvl.TVL_F16, "q8": tvl.TVL_Q8, "q4": tvl.TVL_Q4}
BITS = {"f32": 32, "f16": 16, "q8": 8, "q4": 4}
EPS = 1e-5
DEV = "cuda"


# ------------------------------------------------------------------- the cases
def listed():
    return [
        # one attention projection of the 110M model: the smallest call, bound by its launch
        dict(name="gemv_attn110m_f32", kind="gemv", M=768, K=768, dtype="f32"),
        # key or value projection of a 70B-shaped layer (grouped heads): few, long rows
        dict(name="gemv_kv70b_f16", kind="gemv", M=1024, K=8192, dtype="f16"),
        # the classifier, called by itself after the last layer
        dict(name="gemv_classifier_f32", kind="gemv", M=32000, K=768, dtype="f32"),
        # the FFN's output projection of a 4-bit 7B layer, called by itself
        dict(name="gemv_w2_7b_q4", kind="gemv", M=4096, K=11008, dtype="q4"),
        # the FFN's input step of a 110M layer: RMSNorm, w1 and w3, SwiGLU in one item
        dict(name="item_ffn110m_f32", kind="ffn", M=2048, K=768, dtype="f32"),
        # the attention-input step of an 8-bit 7B layer: wq, wk, wv in one launch
        dict(name="plan_qkv7b_q8", kind="plan", part="qkv", dim=4096, kv=4096, hidden=11008,
             layers=1, vocab=0, dtype="q8", nrhs=1, fused=False),
        # a whole 110M token in one launch, fp32: this repository's headline
        dict(name="token110m_f32", kind="plan", part="all", dim=768, kv=768, hidden=2048,
             layers=12, vocab=32000, dtype="f32", nrhs=1, fused=False),
        # the same token with 4-bit weights
        dict(name="token110m_q4", kind="plan", part="all", dim=768, kv=768, hidden=2048,
             layers=12, vocab=32000, dtype="q4", nrhs=1, fused=False),
        # a whole 7B token with 4-bit weights: the largest launch
        dict(name="token7b_q4", kind="plan", part="all", dim=4096, kv=4096, hidden=11008,
             layers=32, vocab=32000, dtype="q4", nrhs=1, fused=False),
        # one 70B-shaped fp16 layer with RMSNorms and the SwiGLU pair fused
        dict(name="layer70b_fused_f16", kind="plan", part="all", dim=8192, kv=1024, hidden=28672,
             layers=1, vocab=0, dtype="f16", nrhs=1, fused=True),
        # beam search, 4 hypotheses, one attention output projection of a 7B layer
        dict(name="beam4_wo7b_f16", kind="beam", M=4096, K=4096, dtype="f16", nrhs=4),
        # beam search, 8 hypotheses, one 110M layer
        dict(name="beam8_layer110m_f32", kind="plan", part="all", dim=768, kv=768, hidden=2048,
             layers=1, vocab=0, dtype="f32", nrhs=8, fused=False),
    ]


def _size(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi]: half of them whole multiples of 64."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, n // 64 * 64) if rng.random() < 0.5 else n


def draw(rng):
    kind = rng.choice(["gemv", "gemv", "gemv", "ffn", "beam", "beam", "plan", "plan", "plan"])
    if kind != "plan":
        while True:
            M, K = _size(rng, 256, 32000), _size(rng, 256, 28672)
            if M * K <= 150_000_000:
                break
        if kind == "gemv":
            return dict(kind=kind, M=M, K=K, dtype=rng.choice(["f32", "f16", "q8", "q4"]))
        dtype = rng.choice(["f32", "f16"])
        if kind == "ffn":
            return dict(kind=kind, M=M, K=K, dtype=dtype)
        return dict(kind=kind, M=M, K=K, dtype=dtype, nrhs=rng.randint(2, 16))
    option = rng.choice(["plain", "plain", "plain", "fused", "beam"])
    dtype = rng.choice(["f32", "f16", "q8", "q4"] if option == "plain" else ["f32", "f16"])
    part = rng.choice(["qkv", "all", "all"])
    dim = _size(rng, 512, 8192)
    kv = max(64, dim // rng.choice([1, 1, 4, 8]))
    hidden = int(dim * rng.choice([2.67, 2.6875, 3.5])) // 8 * 8
    layer = 2 * dim * (dim + kv) + 3 * dim * hidden
    # at most 3 GB of weights in a launch
    most = max(1, int(3e9 * 8 / BITS[dtype] / layer))
    layers = 1 if part == "qkv" else min(rng.choice([1, 1, 8, 32]), most)
    vocab = 32000 if layers > 1 and rng.random() < 0.5 else 0
    return dict(kind="plan", part=part, dim=dim, kv=kv, hidden=hidden, layers=layers, vocab=vocab,
                dtype=dtype, nrhs=rng.randint(2, 16) if option == "beam" else 1,
                fused=option == "fused")


# ---------------------------------------------------------------- their inputs
def _mats(case):
    """The case's items: (M, K, input, pair, norm) each, `input` naming the x vector
    that items of one step share, `pair` a SwiGLU pair, `norm` a fused RMSNorm."""
    if case["kind"] in ("gemv", "beam"):
        return [(case["M"], case["K"], "x", False, False)]
    if case["kind"] == "ffn":
        return [(case["M"], case["K"], "x", True, True)]
    d, h, kv, fused = case["dim"], case["hidden"], case["kv"], case["fused"]
    out = []
    for l in range(case["layers"]):
        out += [(m, d, f"att{l}", False, fused) for m in (d, kv, kv)]
        if case["part"] == "qkv":
            continue
        out.append((d, d, f"wo{l}", False, False))
        if fused:
            out.append((h, d, f"ffn{l}", True, True))
        else:
            out += [(h, d, f"ffn{l}", False, False)] * 2
        out.append((d, h, f"w2{l}", False, False))
    if case["vocab"]:
        out.append((case["vocab"], d, "final", False, fused))
    return out


def _nrhs(case):
    return case.get("nrhs", 1)


class _Inputs:
    """The items' tensors, drawn one after the other from the seed."""

    def __init__(self, case, seed):
        self.case = case
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(seed)
        self.vecs = {}

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.gen, device=DEV)

    def weights(self, M, K):
        """The matrix in the library's layout (one tensor), and its row stride."""
        dtype = self.case["dtype"]
        ldw = tvl.tvl_row_stride(K, DT[dtype])
        if dtype in ("f32", "f16"):
            t = torch.float32 if dtype == "f32" else torch.float16
            W = torch.zeros(M, ldw, dtype=t, device=DEV)
            W[:, :K] = self.normal(M, K).mul_(0.02)
            return W, ldw
        bits, ng, Mp = BITS[dtype], (K + 63) // 64, (M + 3) // 4 * 4
        w = torch.zeros(M, ng * 64, device=DEV)
        w[:, :K] = self.normal(M, K).mul_(0.02)
        w = w.view(M, ng, 64)
        top = (1 << (bits - 1)) - 1
        scale = (w.abs().amax(2) / top).clamp_min_(1e-30)
        q = torch.round(w / scale.unsqueeze(2)).to(torch.int8).view(M, ng * 64)
        if bits == 4:
            q = (q[:, 0::2] & 15) | (q[:, 1::2] << 4)
        buf = torch.zeros(M * ldw + 4 * Mp * ng, dtype=torch.uint8, device=DEV)
        n = min(ldw, q.shape[1])
        buf[:M * ldw].view(M, ldw)[:, :n] = q[:, :n].view(torch.uint8)
        plane = torch.zeros(Mp, ng, device=DEV)
        plane[:M] = scale
        plane = plane.view(Mp // 4, 4, ng).permute(0, 2, 1).reshape(-1)  # blocks of 4 rows
        buf[M * ldw:] = plane.contiguous().view(torch.uint8)
        return buf, ldw

    def x(self, name, K):
        n = _nrhs(self.case)
        if name not in self.vecs:
            if n == 1:
                self.vecs[name] = self.normal(K)
            else:
                X = torch.zeros(n, (K + 3) // 4 * 4, device=DEV)
                X[:, :K] = self.normal(n, K)
                self.vecs[name] = X
        return self.vecs[name]

    def g(self, name, K):
        if "g" + name not in self.vecs:
            self.vecs["g" + name] = 1 + 0.1 * self.normal(K)
        return self.vecs["g" + name]

    def items(self):
        for M, K, name, pair, norm in _mats(self.case):
            W, ldw = self.weights(M, K)
            W3 = self.weights(M, K)[0] if pair else None
            yield M, K, ldw, W, W3, self.x(name, K), self.g(name, K) if norm else None


def prepare(case, seed):
    mats, n = _mats(case), _nrhs(case)
    y = torch.empty(n * sum(m[0] for m in mats), device=DEV)
    keep, items, at = [y], [], 0
    for M, K, ldw, W, W3, x, g in _Inputs(case, seed).items():
        keep += [W, W3, x, g]
        items.append(dict(W=W, ldw=ldw, x=x, y=y[at:at + n * M], M=M, K=K, dtype=DT[case["dtype"]],
                          op=tvl.TVL_OP_GEMV if W3 is None else tvl.TVL_OP_SWIGLU, W3=W3, g=g,
                          eps=EPS if g is not None else 0.0, nrhs=n,
                          ldx=x.shape[1] if n > 1 else 0, ldy=M if n > 1 else 0))
        at += n * M
    state = dict(kind=case["kind"], keep=keep, y=y)
    if case["kind"] == "plan":
        state["plan"] = tvl.tvl_sweep_plan_create(items)
    elif case["kind"] == "gemv":
        state["args"] = tuple(items[0][k] for k in ("W", "ldw", "dtype", "x", "y", "M", "K"))
    else:
        state["item"] = tvl.item(**items[0])
    return state


def run(state):
    if state["kind"] == "plan":
        state["plan"].run()
    elif state["kind"] == "gemv":
        tvl.tvl_gemv(*state["args"])
    else:
        tvl.tvl_gemv_item(state["item"])
    return state["y"]


# ------------------------------------------------------- what they are held to
def work(case):
    n, bits = _nrhs(case), BITS[case["dtype"]]
    nbytes, flops, seen = 0, 0, set()
    for M, K, name, pair, norm in _mats(case):
        w = M * ((K * bits + 7) // 8) + (4 * M * ((K + 63) // 64) if bits < 16 else 0)
        nbytes += (2 if pair else 1) * w + 4 * n * M
        flops += (2 if pair else 1) * 2 * M * K * n
        if name not in seen:
            seen.add(name)
            nbytes += 4 * K * (n + (1 if norm else 0))
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Products and sums in 32 bits: against 64 bits the cases show 1e-7 to 3e-7 (2-norm),
    # and another order of the sums shows as much.
    return {"rel": 1e-6, "max": 1e-5}


def _dense(case, W, M, K, ldw):
    """The matrix's values in 64 bits."""
    if case["dtype"] in ("f32", "f16"):
        return W[:, :K].double()
    ng, Mp = (K + 63) // 64, (M + 3) // 4 * 4
    codes = W[:M * ldw].view(M, ldw).view(torch.int8)
    if case["dtype"] == "q4":
        codes = torch.stack([(codes << 4) >> 4, codes >> 4], 2).view(M, 2 * ldw)
    plane = W[M * ldw:].view(torch.float32).view(Mp // 4, ng, 4).permute(0, 2, 1).reshape(Mp, ng)
    scale = plane[:M].double().repeat_interleave(64, 1)[:, :K]
    return codes[:, :K].double() * scale


def exact(case, seed):
    n, out = _nrhs(case), []
    for M, K, ldw, W, W3, x, g in _Inputs(case, seed).items():
        v = x.double().view(n, -1)[:, :K]
        if g is not None:
            v = v * g.double() / torch.sqrt((v * v).mean(1, keepdim=True) + EPS)
        a = v @ _dense(case, W, M, K, ldw).t()
        if W3 is not None:
            a = a / (1 + torch.exp(-a)) * (v @ _dense(case, W3, M, K, ldw).t())
        out.append(a.reshape(-1))
    return torch.cat(out)
