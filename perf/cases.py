"""The work that a user of this library has it do, as cases to time and compare.

A case is one pass of a parameter-server program over gradients that are already in device
memory: the encoder of all P compute nodes (or of one node), the decoder on the messages as they
were received, and, in a training program, the model update.  Shapes come from the workloads of
`paper_1803_09877_amd/synth.py` and of the tests, or lie between them.

Fields of a case
  op      "step"   encode all nodes, decode synchronously (mask and status on the host)
          "train"  encode all nodes, decode stream-ordered, apply the update to the parameters
          "node"   one compute node's own encoder on its 2s+1 gradients
  code    "rep" or "cyc"
  P, s    nodes and tolerated adversaries
  d       gradient length
  m       per-sample gradients per unit gradient (B = m P rows)
  wire    cyclic messages: "one" fp32 word, "i8" / "bf16" / "f32" second word, "unpacked"
  liars   adversarial nodes among the received messages
  sigma   standard deviation of the gradients
  stored  projection vector: True = the caller's, False = made inside the decoder
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_1803_09877_amd import binding as B
from paper_1803_09877_amd import synth

DEVICE = "cuda:0"
LO_DTYPE = {"i8": torch.int8, "bf16": torch.bfloat16, "f32": torch.float32}
LO_BYTES = {"one": 0, "unpacked": 0, "i8": 1, "bf16": 2, "f32": 4}
LO_FORMAT = {"i8": B.SECOND_WORD_I8, "bf16": B.SECOND_WORD_BF16, "f32": B.SECOND_WORD_F32}
ATTACKS = ("noise", "signflip", "constant")
LEARNING_RATE = 0.05


def _case(name, op, code, P, s, d, m=1, wire="one", liars=0, sigma=1e-2, stored=False):
    return {"name": name, "op": op, "code": code, "P": P, "s": s, "d": d, "m": m, "wire": wire, "liars": liars,
            "sigma": sigma, "stored": stored}


def listed():
    return [
        # the smallest benchmark workload: a toy model on 15 nodes; launches and latency
        _case("rep_small", "step", "rep", 15, 1, 10_000, liars=1, sigma=1.0),
        # ResNet-18's length on the paper's 45 nodes, reversed-gradient adversaries
        _case("rep_resnet18", "step", "rep", 45, 2, 11_200_000, liars=2),
        # a training step of a small convolutional model, B = 180 on 45 nodes, an odd length, nobody lies
        _case("rep_batch180", "train", "rep", 45, 2, 1_663_371, m=4),
        # a small model on 45 nodes with the cyclic code: the decoder's latency chain
        _case("cyc_small", "step", "cyc", 45, 3, 30_000, wire="i8", liars=3, stored=True),
        # 15 nodes, one word per float
        _case("cyc_p15", "step", "cyc", 15, 2, 4_000_000, liars=2, sigma=1.0, stored=True),
        # the headline: ResNet-50's length on 45 nodes, 5-byte wire, three adversaries
        _case("cyc_headline", "step", "cyc", 45, 3, 25_600_000, wire="i8", liars=3, stored=True),
        # the usual training step: nobody lies, projection made in the decoder, odd length
        _case("cyc_clean_train", "train", "cyc", 45, 3, 1_200_001, wire="i8"),
        # the paper's timing runs: B = 180, s = 5, persistent adversaries
        _case("cyc_batch180", "step", "cyc", 45, 5, 25_600_000, m=4, wire="i8", liars=5),
        # the widest window of the paper's experiments on the most exact wire
        _case("cyc_s7_exact", "step", "cyc", 45, 7, 6_000_000, wire="f32", liars=4, stored=True),
        # a mid-sized model, 6-byte wire, ragged length, one adversary, update applied
        _case("cyc_bf16_train", "train", "cyc", 32, 4, 3_000_003, wire="bf16", liars=1),
        # the code as Section 3 states it: complex messages of real gradients
        _case("cyc_unpacked", "step", "cyc", 15, 2, 1_000_000, wire="unpacked", liars=1, sigma=1.0),
        # one compute node's own encoder in a real deployment
        _case("cyc_node", "node", "cyc", 45, 5, 11_200_000, wire="i8"),
    ]


def draw(rng: random.Random):
    code = rng.choice(("rep", "cyc", "cyc"))
    op = rng.choice(("step", "step", "train", "node"))
    d = int(round(math.exp(rng.uniform(math.log(10_000), math.log(25_600_000)))))
    m = 1 if op == "node" else rng.choice((1, 1, 1, 2, 4, 16))
    if code == "rep":
        s = rng.choice((1, 2, 3, 4))
        P = (2 * s + 1) * rng.randint(2, 45 // (2 * s + 1))
        wire, stored = "one", False
    else:
        s = rng.randint(1, 7)
        P = rng.randint(max(2 * s + 2, 8), 45)
        # one word per float only where it decodes well; the unpacked wire has one word and B = P
        wire = rng.choice(("i8", "i8", "bf16", "f32") + (("one", "unpacked") if P <= 16 and s <= 3 else ()))
        if wire == "unpacked":
            m = 1
        stored = rng.random() < 0.5
    liars = 0 if op == "node" else rng.randint(0, s)
    rows = (2 * s + 1) if op == "node" else P * m
    d = min(d, 180 * 25_600_000 // rows)
    c = _case("", op, code, P, s, d, m, wire, liars, rng.choice((1e-2, 1.0)), stored)
    del c["name"]
    return c


# ---- sizes ---------------------------------------------------------------------------
def _message_len(c):
    if c["code"] == "rep":
        return c["d"]
    return 2 * c["d"] if c["wire"] == "unpacked" else 2 * ((c["d"] + 1) // 2)


def _liars(c, seed):
    """(node, attack) of each adversary: nodes drawn from the seed, in different groups where the
    repetition code has them."""
    rng = random.Random(seed * 7 + 1)
    if c["code"] == "rep":
        r = 2 * c["s"] + 1
        groups = list(range(c["P"] // r))
        rng.shuffle(groups)
        nodes = [groups[i % len(groups)] * r + (i // len(groups)) + rng.randrange(c["s"]) for i in range(c["liars"])]
    else:
        nodes = rng.sample(range(c["P"]), c["liars"])
    return [(j, ATTACKS[i % len(ATTACKS)]) for i, j in enumerate(sorted(set(nodes)))]


def _rows(c):
    return 2 * c["s"] + 1 if c["op"] == "node" else c["P"] * c["m"]


def _gradients(c, seed):
    return synth.make_gradients(_rows(c), c["d"], c["sigma"], seed, device=DEVICE)


def _parameters(c, seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed + 3)
    return torch.randn(synth.padded_len(c["d"]), generator=g, device=DEVICE) * 0.1


def _scale(c):
    return LEARNING_RATE / (c["P"] * c["m"])


# ---- a user's program ----------------------------------------------------------------
def prepare(c, seed):
    """Gradients, plan, output slabs, and the messages as received (some of them rewritten)."""
    st = {"case": c}
    code = B.CODE_REPETITION if c["code"] == "rep" else B.CODE_CYCLIC
    plan = B.Plan(code, c["P"], c["s"], c["d"])
    if c["wire"] == "unpacked":
        plan.set_wire(B.WIRE_UNPACKED)
    if c["wire"] in LO_DTYPE:
        plan.set_second_word(LO_FORMAT[c["wire"]])
    if c["code"] == "cyc":
        plan.set_projection_seed(seed)
    plan.prepare()
    st["plan"] = plan
    st["G"] = _gradients(c, seed)
    mlen = _message_len(c)
    ld = synth.padded_len(mlen)
    two = c["wire"] in LO_DTYPE
    if c["op"] == "node":
        st["node"] = seed % c["P"]
        st["Z"] = torch.zeros(ld, device=DEVICE)
        st["Zlo"] = torch.zeros(ld, dtype=LO_DTYPE[c["wire"]], device=DEVICE) if two else None
        return st
    st["Z"] = torch.zeros((c["P"], ld), device=DEVICE)
    st["Zlo"] = torch.zeros((c["P"], ld), dtype=LO_DTYPE[c["wire"]], device=DEVICE) if two else None
    _encode(st)
    st["R"] = st["Z"].clone()
    st["Rlo"] = st["Zlo"].clone() if two else None
    synth.apply_attacks(st["R"], mlen, _liars(c, seed), seed)
    st["u"] = torch.zeros(synth.padded_len(c["d"]), device=DEVICE)
    st["f"] = synth.make_projection(mlen // 2, seed, device=DEVICE) if c["stored"] and c["code"] == "cyc" else None
    if c["op"] == "train":
        st["w"] = _parameters(c, seed)
        st["mask"] = torch.zeros(4, dtype=torch.int64, device=DEVICE)
        st["status"] = torch.zeros(1, dtype=torch.int32, device=DEVICE)
    return st


def _encode(st):
    c, plan = st["case"], st["plan"]
    if st["Zlo"] is not None:
        if c["m"] > 1:
            plan.encode_samples_wide(st["G"], st["Z"], st["Zlo"])
        else:
            plan.encode_wide(st["G"], st["Z"], st["Zlo"])
    elif c["m"] > 1:
        plan.encode_samples(st["G"], st["Z"])
    else:
        plan.encode(st["G"], st["Z"])


def run(st):
    c, plan = st["case"], st["plan"]
    mlen = _message_len(c)
    if c["op"] == "node":
        if st["Zlo"] is not None:
            plan.encode_node_wide(st["node"], st["G"], st["Z"], st["Zlo"])
            return {"message": st["Z"][:mlen], "second": st["Zlo"][:mlen]}
        plan.encode_node(st["node"], st["G"], st["Z"])
        return {"message": st["Z"][:mlen]}
    _encode(st)
    out = {"messages": st["Z"][:, :mlen], "sum": st["u"][:c["d"]]}
    if st["Zlo"] is not None:
        out["second"] = st["Zlo"][:, :mlen]
    if c["op"] == "train":
        if c["code"] == "rep":
            plan.decode_repetition_async(st["R"], st["u"], st["mask"], st["status"])
        elif st["Rlo"] is not None:
            plan.decode_cyclic_wide_async(st["R"], st["Rlo"], st["f"], st["u"], st["mask"], st["status"])
        else:
            plan.decode_cyclic_async(st["R"], st["f"], st["u"], st["mask"], st["status"])
        B.draco_apply_update(st["w"], st["u"], c["d"], _scale(c))
        out["params"] = st["w"][:c["d"]]
        out["mask"], out["status"] = st["mask"], st["status"]
        return out
    if c["code"] == "rep":
        mask, status = plan.decode_repetition(st["R"], st["u"])
    elif st["Rlo"] is not None:
        mask, status = plan.decode_cyclic_wide(st["R"], st["Rlo"], st["f"], st["u"])
    else:
        mask, status = plan.decode_cyclic(st["R"], st["f"], st["u"])
    out["mask"], out["status"] = mask, status
    return out


def work(c):
    """Each input read once, each output written once."""
    P, s, d, mlen = c["P"], c["s"], c["d"], _message_len(c)
    r = 2 * s + 1
    per = 4 + LO_BYTES[c["wire"]]
    if c["op"] == "node":
        flops = r * d if c["code"] == "rep" else mlen // 2 * (4 * r + 8)
        return {"bytes": 4 * r * d + per * mlen, "flops": flops}
    bytes_ = 4 * P * c["m"] * d + per * P * mlen          # encode
    bytes_ += per * P * mlen + 4 * d                      # decode: every message once, the sum
    if c["stored"] and c["code"] == "cyc":
        bytes_ += 4 * (mlen // 2)
    if c["op"] == "train":
        bytes_ += 12 * d
    if c["code"] == "rep":
        flops = P * c["m"] * d + P // r * d
    else:
        flops = P * (c["m"] - 1) * d + mlen // 2 * P * (4 * r + 8) + mlen // 2 * P * 12
    return {"bytes": bytes_, "flops": flops}


def tolerance(c):
    """About four times what the library is from `exact` (or from exact's value taken through the
    same rounding), over the listed sizes and a few drawn ones.
    Repetition code: fp32 sums of up to 144 numbers, 1.1e-7.  Cyclic code: fp64 sums rounded once
    to fp32, 2.5e-8, equal but for 1e-6 of the values, which straddle a rounding boundary.  The
    second word of the two-word wires holds what that rounding left, so the last bits of the fp64
    sum show in it: an 8-bit code differs by one step in 1.4e-4 of the places (and the decoded sum
    by 4e-7), a 16- or 32-bit second word by 8e-4 of itself, by its whole size where the first word
    straddles a boundary."""
    if c["code"] == "rep":
        return {"rel": 1e-6, "max": 2e-5}
    if c["wire"] == "i8":
        return {"rel": 2e-6, "max": 4e-5, "differ": 6e-4}
    if c["wire"] in ("bf16", "f32"):
        return {"rel": 3.3e-3, "max": 0.99}
    return {"rel": 2e-7, "max": 2e-6}


# ---- the same in 64 bits, without the library ----------------------------------------
def _weights(P, s):
    """W[k][j] = P^-1/2 prod over the nodes m that do not hold gradient k of (w^j - w^m),
    w = exp(2 pi i / P); node j holds gradients j .. j+2s (mod P)."""
    ang = 2 * np.pi * np.arange(P, dtype=np.longdouble) / P
    w = np.cos(ang) + 1j * np.sin(ang)
    out = np.zeros((P, P), dtype=np.clongdouble)
    for k in range(P):
        outside = [m for m in range(P) if (k - m) % P > 2 * s]
        for j in range(P):
            if (k - j) % P <= 2 * s:
                out[k, j] = np.prod(w[j] - w[outside]) / np.sqrt(np.longdouble(P))
    return torch.from_numpy(out.astype(np.complex128)).to(DEVICE)


def exact(c, seed):
    P, s, d, m, mlen = c["P"], c["s"], c["d"], c["m"], _message_len(c)
    r = 2 * s + 1
    G = _gradients(c, seed)
    node = seed % P if c["op"] == "node" else None
    rows = 1 if node is not None else P
    Z = torch.zeros((rows, mlen), dtype=torch.float64, device=DEVICE)
    u = torch.zeros(d, dtype=torch.float64, device=DEVICE)
    W = _weights(P, s) if c["code"] == "cyc" else None
    step = 1 << 20
    for a in range(0, d, step):
        b = min(d, a + step)
        g = G[:, a:b].double()
        if node is None:
            g = g.reshape(P, m, b - a).sum(1)
            u[a:b] = g.sum(0)
        if c["code"] == "rep":
            z = g.reshape(-1, r, b - a).sum(1)
            Z[:, a:b] = z if node is not None else z.repeat_interleave(r, 0)
            continue
        Wc = W if node is None else W[[(node + t) % P for t in range(r)], node].reshape(r, 1)
        if c["wire"] == "unpacked":
            z = torch.view_as_real(torch.mm(Wc.t().contiguous(), g.to(torch.complex128)))
            Z[:, 2 * a:2 * b] = z.reshape(rows, -1)
        else:
            if (b - a) % 2:
                g = torch.cat([g, torch.zeros_like(g[:, :1])], 1)
            gc = torch.complex(g[:, 0::2].contiguous(), g[:, 1::2].contiguous())
            Z[:, a:a + g.shape[1]] = torch.view_as_real(torch.mm(Wc.t().contiguous(), gc)).reshape(rows, -1)
    if node is not None:
        out = {"message": Z.reshape(-1)}
        if c["wire"] in LO_DTYPE:
            out["second"] = None
        return out
    out = {"messages": Z, "sum": u}
    if c["wire"] in LO_DTYPE:
        out["second"] = None
    bad = [j for j, _ in _liars(c, seed)]
    if c["op"] == "train":
        words = np.zeros(4, dtype=np.uint64)
        for j in bad:
            words[j >> 6] |= np.uint64(1) << np.uint64(j & 63)
        out["params"] = _parameters(c, seed)[:d].double() - _scale(c) * u
        out["mask"], out["status"] = torch.from_numpy(words.view(np.int64).copy()), torch.zeros(1, dtype=torch.int32)
    else:
        mask = np.zeros(P, dtype=bool)
        mask[bad] = True
        out["mask"], out["status"] = mask, 0
    return out
