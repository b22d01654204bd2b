"""Measured work: what programs built on this library have it do, through its public calls.

A program of this library is the server side of encrypted inference (plus the making of fresh ciphertexts on the device).
It holds a context, switching keys, layer weights and workspaces, and calls the operations below on batches of
ciphertexts.  The listed cases are the shapes of the repository's presets and benchmark, from sixteen small products to
whole batches at N = 2^16; `draw` gives others between them: ring degrees 2^12 .. 2^16, any level, batches from one
ciphertext on, odd sizes.

Ciphertexts, keys and public keys are uniform residues: that is how RLWE ciphertexts are distributed, and no kernel
branches on their values.  Slot values are uniform on [-1, 1], layer weights N(0, 0.05^2) rounded at the scale of the
dropped prime, as in the repository's workloads.

All outputs are residues modulo the context's primes, whole numbers that any correct implementation of the call
reproduces word for word, so every tolerance is "exact".  (The encoder rounds real numbers; its rounded coefficients are
whole numbers too, and a different rounding would change every word of a transformed limb.)
"""
import numpy as np
import torch

from paper_1911_11377_amd import activation, ckksmi, packed
from paper_1911_11377_amd import workloads as wl

DEV = "cuda:0"

# ring parameters: (primes, prime bits, special primes, special bits, primes per key-switching digit)
CHAINS = {
    "tiny": (3, 40, 1, 41, 1),       # the smallest workload's chain
    "short": (8, 50, 1, 51, 1),      # products and rotations at N = 2^14
    "network": (11, 50, 3, 51, 3),   # one image through a small network
    "conv": (16, 50, 0, 51, 1),      # convolution layer without key switching
    "deep": (24, 50, 3, 51, 3),      # activations at depth
}


def listed():
    return [
        # 16 small ciphertext products with relinearisation and rescale: the latency of the composite call
        {"name": "product_2e12_b16", "op": "product", "logN": 12, "chain": "tiny", "level": 3, "batch": 16},
        # the same call on a server's batch of mid-size ciphertexts
        {"name": "product_2e14_b256", "op": "product", "logN": 14, "chain": "short", "level": 8, "batch": 256},
        # the headline: products at N = 2^16 in full depth
        {"name": "product_2e16_b64", "op": "product", "logN": 16, "chain": "deep", "level": 24, "batch": 64},
        # slot rotations of a ragged batch, every ciphertext by one of 8 offsets, one level below the top
        {"name": "rotate_2e14_b131", "op": "rotate", "logN": 14, "chain": "short", "level": 7, "batch": 131, "keys": 8},
        # all 8 rotations of each ciphertext from one shared decomposition (the first half of a packed matrix product)
        {"name": "rotations_shared_2e14_b32", "op": "rotate_shared", "logN": 14, "chain": "short", "level": 8, "batch": 32, "keys": 8},
        # degree-3 polynomial activation of an odd number of ciphertexts, last digit of one prime
        {"name": "activation_2e16_b21", "op": "activation", "logN": 16, "chain": "deep", "level": 22, "batch": 21},
        # convolution layer 3 -> 32, 5x5, stride 2, on per-pixel ciphertexts of 16384 images: two of its 14 output rows,
        # multiply-accumulate and rescale, as a layer that exceeds the memory is walked strip by strip
        {"name": "conv_2e15_rows2", "op": "conv", "logN": 15, "chain": "conv", "level": 16, "cin": 3, "size": 32, "cout": 32, "kernel": 5, "stride": 2,
         "pad": 0, "rows": 2},
        # fully connected layer 3136 -> 256 (the first one after the convolutions of the 2^16 network), with its rescale
        {"name": "fc_2e14_3136x256", "op": "fc", "logN": 14, "chain": "short", "level": 8, "fin": 3136, "fout": 256},
        # plain limb transforms, evaluation form and back
        {"name": "ntt_2e16_3456", "op": "ntt", "logN": 16, "chain": "deep", "level": 24, "batch": 144, "inverse": False},
        {"name": "intt_2e15_2000", "op": "ntt", "logN": 15, "chain": "conv", "level": 16, "batch": 125, "inverse": True},
        # fresh ciphertexts made on the device: randomness, encoding of real slots, encryption
        {"name": "fresh_2e16_b64", "op": "fresh", "logN": 16, "chain": "deep", "level": 24, "batch": 64},
        # one image, one dense layer in the rotation-packed layout with baby and giant steps: a single ciphertext, latency
        {"name": "packed_layer_2e14_64", "op": "packed", "logN": 14, "chain": "short", "level": 8, "size": 64},
    ]


# one draw costs at most about what the headline batch does: words that cross a key switch, or a layer's word products
MAX_KS_WORDS = 64 * (8 * 27 + 6 * 24) << 16
MAX_MAC_WORDS = 32 * 28 * 75 * 32 << 15


def _logint(rng, lo, hi):
    """a whole number between lo and hi, spread over its logarithm"""
    return min(hi, max(lo, int(round(np.exp(rng.uniform(np.log(lo), np.log(hi + 0.5)))))))


def draw(rng):
    op = rng.choice(["product", "product", "rotate", "rotate_shared", "activation", "conv", "fc", "ntt", "ntt", "fresh", "packed"])
    logN = rng.randint(12, 16)
    if op in ("product", "rotate", "rotate_shared", "activation", "ntt", "fresh"):
        chain = rng.choice(["tiny", "short", "network", "deep"])
        nq, _, k, _, alpha = CHAINS[chain]
        lo = {"activation": 3, "product": 2}.get(op, 1)
        level = rng.randint(lo, nq)
        beta = -(-level // alpha)
        per = (beta * (level + k) + 6 * level) << logN
        case = {"op": op, "logN": logN, "chain": chain, "level": level}
        if op == "rotate":
            case["keys"] = rng.randint(1, 8)
        if op == "rotate_shared":
            case["keys"] = rng.randint(2, 24)
            per *= case["keys"]
        if op == "activation":
            per *= 3
        if op == "ntt":
            case["inverse"] = rng.random() < 0.5
            per = 2 * level << logN
        case["batch"] = _logint(rng, 1, max(1, min(512, MAX_KS_WORDS // (2 * per))))
        return case
    if op == "packed":
        # (the period is a power of two whatever the matrix size)
        return {"op": op, "logN": rng.randint(12, 14), "chain": rng.choice(["short", "network"]), "level": rng.randint(3, 8), "size": _logint(rng, 10, 128)}
    chain = rng.choice(["short", "conv"])
    level = rng.randint(2, CHAINS[chain][0])
    logN = rng.randint(12, 15)
    if op == "fc":
        case = {"op": op, "logN": logN, "chain": chain, "level": level, "fin": _logint(rng, 20, 1600), "fout": _logint(rng, 8, 256)}
        while (case["fin"] * case["fout"] * 2 * level << logN) > MAX_MAC_WORDS:
            case["fin"] = max(8, case["fin"] // 2)
            case["fout"] = max(8, case["fout"] * 2 // 3)
        return case
    kernel, stride = rng.choice([3, 5]), rng.randint(1, 2)
    case = {"op": op, "logN": logN, "chain": chain, "level": level, "cin": rng.randint(1, 16), "size": rng.randint(6, 20), "cout": rng.randint(8, 48),
            "kernel": kernel, "stride": stride, "pad": rng.randint(0, kernel // 2), "rows": rng.randint(1, 2)}
    while _conv_words(case) > MAX_MAC_WORDS:
        case["cin"] = max(1, case["cin"] // 2)
        case["cout"] = max(8, case["cout"] * 2 // 3)
        case["level"] = max(2, case["level"] - 1)
    return case


def _conv_words(case):
    wo = (case["size"] + 2 * case["pad"] - case["kernel"]) // case["stride"] + 1
    return case["cout"] * case["rows"] * wo * case["cin"] * case["kernel"] ** 2 * 2 * case["level"] << case["logN"]


# ------------------------------------------------------------------------------------------------------------ preparation
def _context(case):
    nq, qb, k, sb, alpha = CHAINS[case["chain"]]
    return ckksmi.Context(case["logN"], nq, qb, k, sb, alpha, device=0)


def _residues(ctx, index, lead, gen):
    """[*lead][len(index)][N], limb x uniform on [0, modulus[index[x]])"""
    out = torch.empty(tuple(lead) + (len(index), ctx.N), dtype=torch.int64, device=DEV)
    for x, i in enumerate(index):
        out[..., x, :] = torch.randint(0, ctx.moduli[i], tuple(lead) + (ctx.N,), dtype=torch.int64, device=DEV, generator=gen)
    return out


def _key(ctx, gen):
    return _residues(ctx, range(ctx.T), (ctx.beta_top, 2), gen)


def _words(*shape):
    return torch.empty(shape, dtype=torch.int64, device=DEV)


def _ws(nbytes):
    return _words(-(-int(nbytes) // 8) + 2)


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    host = np.random.default_rng([int(seed), 17])
    ctx = _context(case)
    op, L, N = case["op"], case["level"], ctx.N
    s = {"case": case, "ctx": ctx}
    if op == "product":
        B = case["batch"]
        s["a"], s["b"] = _residues(ctx, range(L), (B, 2), gen), _residues(ctx, range(L), (B, 2), gen)
        s["evk"], s["out"] = _key(ctx, gen), _words(B, 2, L - 1, N)
        s["ws"] = _ws(ctx.workspace_bytes(ckksmi.OP_HMUL_RELIN_RESCALE, L, B))
    elif op == "rotate":
        B = case["batch"]
        s["a"], s["out"] = _residues(ctx, range(L), (B, 2), gen), _words(B, 2, L, N)
        offsets = [int(x) for x in host.choice(np.arange(1, N // 2), size=case["keys"], replace=False)]
        for r in offsets:
            ctx.galois_key_register(r, _key(ctx, gen))
        s["rot"] = [offsets[int(i)] for i in host.integers(0, len(offsets), size=B)]
        s["ws"] = _ws(ctx.workspace_bytes(ckksmi.OP_ROTATE, L, B))
    elif op == "rotate_shared":
        B = case["batch"]
        s["a"], s["out"] = _residues(ctx, range(L), (B, 2), gen), _words(B, case["keys"], 2, L, N)
        s["rot"] = [int(x) for x in host.choice(np.arange(1, N // 2), size=case["keys"], replace=False)]
        for r in s["rot"]:
            ctx.galois_key_register(r, _key(ctx, gen))
        s["ws"] = _ws(ctx.rotate_hoisted_workspace_bytes(L, B, case["keys"]))
    elif op == "activation":
        B = case["batch"]
        s["a"], s["evk"], s["out"] = _residues(ctx, range(L), (B, 2), gen), _key(ctx, gen), _words(B, 2, L - 2, N)
        bits = CHAINS[case["chain"]][1]
        s["consts"] = activation.poly3_constants(ctx.q, L, 2.0 ** (bits - 1))
        s["ws"] = _ws(activation.workspace_bytes(ctx, L, B))
    elif op in ("conv", "fc"):
        if op == "conv":
            C, H, K, S, P, R, O = (case[x] for x in ("cin", "size", "kernel", "stride", "pad", "rows", "cout"))
            wo = (H + 2 * P - K) // S + 1
            s["wo"], s["rows"] = wo, min(R, wo)
            # the strip: the first output rows and the image rows they need
            s["in_rows"] = min(H, (s["rows"] - 1) * S - P + K)
            n_in, n_out, taps = C * s["in_rows"] * H, O * s["rows"] * wo, C * K * K
            ws = ctx.conv2d_workspace_bytes(C, O, K, K, L)
        else:
            n_in, n_out, taps, O = case["fin"], case["fout"], case["fin"], case["fout"]
            ws = ctx.conv2d_workspace_bytes(n_in, O, 1, 1, L)
        s["x"] = _residues(ctx, range(L), (n_in, 2), gen)
        w = torch.randn((O, taps), dtype=torch.float64, device=DEV, generator=gen) * 0.05
        s["w"] = torch.round(w * float(ctx.q[L - 1])).to(torch.int64)
        s["mac"], s["out"], s["n_out"] = _words(n_out, 2, L, N), _words(n_out, 2, L - 1, N), n_out
        s["ws"], s["ws_rescale"] = _ws(ws), _ws(ctx.workspace_bytes(ckksmi.OP_RESCALE, L, min(n_out, 256)))
    elif op == "ntt":
        s["x"] = _residues(ctx, range(L), (case["batch"],), gen)
    elif op == "fresh":
        B = case["batch"]
        s["re"] = torch.rand((B, N // 2), dtype=torch.float64, device=DEV, generator=gen) * 2 - 1
        s["pk"] = _residues(ctx, range(ctx.n_q), (2,), gen)
        s["small"], s["pt"], s["out"] = [_words(B, N) for _ in range(3)], _words(B, L, N), _words(B, 2, L, N)
        s["seed"], s["scale"] = int(seed), 2.0 ** 40 if CHAINS[case["chain"]][1] >= 50 else 2.0 ** 30
        s["ws"] = _ws(max(B * N * 16, 3 * L * N * 8 * B))
    elif op == "packed":
        s["x"] = _residues(ctx, range(L), (1, 2), gen)
        W = wl.weights_float((case["size"], case["size"]), int(seed), "packed")

        def to_dev(arr):
            return torch.from_numpy(np.ascontiguousarray(arr).view(np.int64)).to(DEV)

        def encode_batch(vecs, scale, level):
            pts = _words(vecs.shape[0], level, N)
            ctx.encode_device(torch.from_numpy(np.ascontiguousarray(vecs)).to(DEV), None, scale, level, vecs.shape[0], pts, _ws(vecs.shape[0] * N * 16))
            return pts

        n = packed.square_pad(W).shape[0]
        s["plan"] = packed.plan_bsgs(ctx, W, n, L, to_dev, encode_batch=encode_batch)
        for r in s["plan"].rotation_offsets():
            ctx.galois_key_register(r, _key(ctx, gen))
        s["out"], s["ws"] = _words(1, 2, L - 1, N), _ws(packed.bsgs_workspace_bytes(ctx, s["plan"]))
    else:
        raise ValueError(op)
    return s


# ------------------------------------------------------------------------------------------------------------ one pass
def run(s):
    c, ctx = s["case"], s["ctx"]
    op, L = c["op"], c["level"]
    if op == "product":
        ctx.hmul_relin_rescale(s["a"], s["b"], s["evk"], s["out"], L, c["batch"], s["ws"])
    elif op == "rotate":
        ctx.rotate(s["a"], s["rot"], s["out"], L, c["batch"], s["ws"])
    elif op == "rotate_shared":
        ctx.rotate_hoisted(s["a"], s["rot"], s["out"], L, c["batch"], s["ws"])
    elif op == "activation":
        activation.poly3(ctx, s["a"], s["evk"], s["out"], L, c["batch"], s["consts"], s["ws"])
    elif op == "conv":
        ctx.conv2d_mac_rows(s["x"], s["w"], c["cin"], c["size"], c["size"], c["cout"], c["kernel"], c["kernel"], c["stride"], c["pad"], 0, s["in_rows"], 0,
                            s["rows"], s["mac"], L, s["ws"])
        ctx.rescale(s["mac"], s["out"], L, s["n_out"], s["ws_rescale"])
    elif op == "fc":
        ctx.fc_mac(s["x"], s["w"], c["fin"], c["fout"], s["mac"], L, s["ws"])
        ctx.rescale(s["mac"], s["out"], L, s["n_out"], s["ws_rescale"])
    elif op == "ntt":
        # in place: a repeated pass transforms the words that the one before left, which are residues again
        (ctx.intt if c["inverse"] else ctx.ntt)(s["x"], range(L), c["batch"])
        return s["x"]
    elif op == "fresh":
        B = c["batch"]
        ctx.sample_device(0, 3.2, s["seed"], 0, B, s["small"][0])
        ctx.sample_device(1, 3.2, s["seed"], B, B, s["small"][1])
        ctx.sample_device(1, 3.2, s["seed"], 2 * B, B, s["small"][2])
        ctx.encode_device(s["re"], None, s["scale"], L, B, s["pt"], s["ws"])
        ctx.encrypt_device(s["pk"], s["pt"], s["small"][0], s["small"][1], s["small"][2], L, B, s["out"], s["ws"])
    elif op == "packed":
        packed.linear_transform_bsgs(ctx, s["x"], s["plan"], s["out"], s["ws"])
    return s["out"]


# ------------------------------------------------------------------------------------------------------------ what a pass needs
def _butterflies(logN, limbs):
    """multiply-adds of `limbs` transforms"""
    return limbs * (logN << (logN - 1))


def _key_switch(c, polys, level=None):
    """(limb transforms, other modular multiply-adds per coefficient) of key-switching `polys` polynomials and dividing by the special primes"""
    nq, _, k, _, alpha = CHAINS[c["chain"]]
    L = level or c["level"]
    beta, E = -(-L // alpha), L + k
    transforms = L + beta * E - L + 2 * k + 2 * L
    others = alpha * (beta * E - L) + 2 * beta * E + 2 * k * L + 2 * L
    return polys * transforms, polys * others


def work(case):
    """Inputs once, outputs once (8 bytes a word); a modular multiply-add counts as two operations."""
    c = case
    op, L, N = c["op"], c["level"], 1 << c["logN"]
    nq, _, k, _, alpha = CHAINS[c["chain"]]
    beta = -(-L // alpha)
    key = beta * 2 * (L + k)
    B = c.get("batch", 1)
    if op == "product":
        t, m = _key_switch(c, B)
        limbs, t, m = B * (4 * L + 2 * (L - 1)) + key, t + B * 2 * L, m + B * (4 * L + 2 * 2 * L)
    elif op == "rotate":
        t, m = _key_switch(c, B)
        limbs = B * 4 * L + key * min(B, c["keys"])
    elif op == "rotate_shared":
        R, E = c["keys"], L + k
        t = B * (L + beta * E - L) + B * R * (2 * k + 2 * L)
        m = B * alpha * (beta * E - L) + B * R * (2 * beta * E + 2 * k * L + 2 * L)
        limbs = B * 2 * L * (1 + R) + key * R
    elif op == "activation":
        t1, m1 = _key_switch(c, B)
        t2, m2 = _key_switch(c, B, L - 1)
        t, m = t1 + t2 + B * 8 * L, m1 + m2 + B * 20 * L
        limbs = B * (2 * L + 2 * (L - 2)) + key
    elif op in ("conv", "fc"):
        if op == "conv":
            wo = (c["size"] + 2 * c["pad"] - c["kernel"]) // c["stride"] + 1
            rows = min(c["rows"], wo)
            n_in = c["cin"] * min(c["size"], (rows - 1) * c["stride"] - c["pad"] + c["kernel"]) * c["size"]
            n_out, taps = c["cout"] * rows * wo, c["cin"] * c["kernel"] ** 2
        else:
            n_in, n_out, taps = c["fin"], c["fout"], c["fin"]
        t, m = n_out * 2 * L, n_out * 2 * (taps * L + 2 * (L - 1))
        limbs = n_in * 2 * L + n_out * 2 * (L - 1)
    elif op == "ntt":
        t, m, limbs = B * L, 0, B * 2 * L
    elif op == "fresh":
        t, m = B * 4 * L + 2 * B, B * 2 * L
        limbs = B * 2 * L + B // 2 + 2 * L
    else:
        n = 1
        while n < c["size"]:
            n *= 2
        baby = packed.bsgs_baby(n)
        giant = n // baby
        t, m = _key_switch(c, baby + giant - 2)
        limbs = 2 * L + 2 * (L - 1) + (baby + giant - 2) * key + n * L
        m += n * 2 * L
    return {"bytes": 8.0 * limbs * N, "flops": 2.0 * (_butterflies(c["logN"], t) + m * N)}


def tolerance(case):
    return "exact"


def exact(case, seed):
    # whole numbers, compared word for word: there is no error to measure
    return None
