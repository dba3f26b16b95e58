"""The work that users of this library have it do, as cases for timing: the obfuscated projection of one batch
(draw A, mix, project, unmix) from decode-shaped batches to whole prefill layers, in float and bf16, for every kind of
A, with A drawn on the spot or ahead of the data.

  listed()              the cases
  draw(rng)             one more case of the same ranges
  prepare(case, seed)   what a program holds before the call: hidden states, weights, a context sized for the shape
  run(state)            one pass through the public entry points; its outputs
  work(case)            bytes and operations one pass cannot do without
  tolerance(case)       how far another correct implementation at the same precision may be off
"""
import math

import torch

from paper_2603_05035_amd import binding as g

KINDS = {"orthogonal": g.GELO_ORTHOGONAL, "gaussian": g.GELO_GAUSSIAN, "conditioned": g.GELO_CONDITIONED,
         "structured": g.GELO_STRUCTURED, "blocks": g.GELO_BLOCK_ORTHOGONAL, "reflectors": g.GELO_REFLECTOR_PRODUCT}
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
SHIELD_SCALE = 10.0          # shield rows: 10 x the median row norm
COND_MAX = 1e3               # acceptance bound of the gaussian kind
MAX_ATTEMPTS = 64


def _case(name, call, kind, dtype, n_data, k_shield, d, p, layers=1):
    c = {"call": call, "kind": kind, "dtype": dtype, "n_data": n_data, "k_shield": k_shield, "d": d, "p": p, "layers": layers}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest whole step there is in the repository: a 16-token float batch of a toy layer; latency and launches
        _case("tiny_f32", "step", "orthogonal", "f32", 16, 2, 64, 192),
        # one decode layer (64 sequences, 4 shield rows) inside a captured or allocation-free serving loop
        _case("decode_static", "static", "orthogonal", "bf16", 64, 4, 4096, 12288),
        # one decode step of a 32-layer model: the 32 matrices of the step drawn by one call, then layer after layer
        _case("decode_sweep", "ahead", "orthogonal", "bf16", 64, 4, 4096, 12288, 32),
        # a float batch of odd size through the generic shapes: rows that fill no tile, widths that are no power of two
        _case("ragged_f32", "step", "orthogonal", "f32", 517, 26, 776, 1544),
        # float layer with the paper's non-orthogonal A, redrawn until its condition number is acceptable
        _case("gaussian_f32", "step", "gaussian", "f32", 512, 0, 4096, 12288),
        # bf16 prefill of one layer with everything on the critical path: A drawn when the batch arrives
        _case("prefill_step", "step", "orthogonal", "bf16", 2048, 102, 4096, 12288),
        # bf16 prefill of 32 layers with A drawn ahead: one call draws all matrices, the layers then only mix / project / unmix
        _case("prefill_ahead", "ahead", "orthogonal", "bf16", 2048, 102, 4096, 12288, 32),
        # the prefill layer with A as a product of directly drawn reflectors
        _case("prefill_reflectors", "step", "reflectors", "bf16", 2048, 102, 4096, 12288),
        # the prefill layer with dense mixing inside blocks of 256 rows
        _case("prefill_blocks", "step", "blocks", "bf16", 2048, 102, 4096, 12288),
        # gate and up projections of the MLP in one, with the structured A: the widest product of the repository's layers
        _case("mlp_structured", "step", "structured", "bf16", 2048, 102, 4096, 22016),
        # the prefill layer with the 8-bit projection: weight quantised once, A drawn ahead, three calls per batch
        _case("prefill_fp8", "fp8", "orthogonal", "bf16", 2048, 102, 4096, 12288),
        # an odd layer of the 32-layer sweep (8 sequences x 512 tokens): dense non-orthogonal A and its inverse
        _case("sweep_conditioned", "step", "conditioned", "bf16", 4096, 0, 4096, 12288),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _log_multiple(rng, lo, hi, step):
    return max(step, round(_log_int(rng, lo, hi) / step) * step)


def draw(rng):
    """One more case: the call and the kind by how often they are used, rows, widths and shields over their ranges."""
    call = rng.choice(["step"] * 5 + ["ahead"] * 2 + ["static", "fp8"])
    if call == "step":
        kind = rng.choice(["orthogonal", "orthogonal", "conditioned", "gaussian", "structured", "blocks", "reflectors"])
    elif call == "ahead":
        kind = rng.choice(["orthogonal", "orthogonal", "blocks", "reflectors"])
    else:
        kind = "orthogonal"
    # A redrawn for its condition number only makes sense in float: bf16 results would be off by kappa(A) roundings
    dtype = "bf16" if call == "fp8" else "f32" if kind == "gaussian" else rng.choice(["bf16", "bf16", "bf16", "f32"])
    most = 122 if call == "static" else 512 if kind == "gaussian" else 2048 if call == "ahead" else 4096
    n_data = _log_int(rng, 1 if call == "static" else 8, most)
    k_shield = 0 if kind == "gaussian" or rng.random() < 0.25 else max(1, round(0.05 * n_data))
    d = _log_multiple(rng, 128, 11008, 128) if call == "fp8" else _log_multiple(rng, 64, 11008, 8)
    p = _log_multiple(rng, 64, 22016, 8)
    while d * p > 4096 * 22016:
        p = _log_multiple(rng, 64, 22016, 8)
    layers = 1
    if call == "ahead":
        n = n_data + k_shield
        room = 32 * min((2150 / n) ** 2, 4096 * 12288 / (d * p), 1.0)
        layers = max(2, min(rng.randint(2, 32), int(room)))
    return _case(None, call, kind, dtype, n_data, k_shield, d, p, layers)


class _State:
    """Inputs, outputs and the context of one case; gives the context back when it is dropped."""

    ctx = None

    def __del__(self):
        if self.ctx is not None:
            g.gelo_destroy(self.ctx)
            self.ctx = None


def _hidden(gen, rows, d, dtype):
    """N(0, 1) with eight channels of twenty times the scale, as the activations of language models have them."""
    H = torch.randn((rows, d), generator=gen, device="cuda", dtype=torch.float32)
    cols = torch.randperm(d, generator=gen, device="cuda")[:min(8, d)]
    H[:, cols] *= 20.0
    return H.to(dtype)


def prepare(case, seed):
    s = _State()
    s.case = dict(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype, kind = DTYPES[case["dtype"]], KINDS[case["kind"]]
    n_data, k, d, p, layers = (case[x] for x in ("n_data", "k_shield", "d", "p", "layers"))
    n = n_data + k
    s.kind, s.k, s.code = kind, k, g.GELO_BF16 if case["dtype"] == "bf16" else g.GELO_F32
    s.H = [_hidden(gen, n_data, d, dtype) for _ in range(layers)]
    s.W = [(torch.randn((d, p), generator=gen, device="cuda", dtype=torch.float32) * 0.02).to(dtype) for _ in range(layers)]
    s.U = torch.empty((n, d), dtype=dtype, device="cuda")
    s.Y = torch.empty((n, p), dtype=dtype, device="cuda")
    s.Z = [torch.empty((n_data, p), dtype=dtype, device="cuda") for _ in range(layers)]
    # batch ids are replayed so that a pass can be repeated; every other part of a call is what a serving program gets
    s.ctx = g.gelo_create(0, seed, allow_batch_reuse=True)
    if case["call"] != "static":
        g.gelo_reserve(s.ctx, kind, s.code, n_data, k, d, p, max_attempts=MAX_ATTEMPTS, mixings=layers)
    if case["call"] == "fp8":
        s.Wq = g.gelo_prepare_weight_fp8(s.ctx, s.W[0])
        s.mixing = g.gelo_sample_mixing(s.ctx, kind, n_data, k, d, s.code, batch_id=1)
    return s


def run(s):
    call = s.case["call"]
    if call == "step":
        g.gelo_qkv_forward(s.ctx, s.kind, s.H[0], s.W[0], s.Z[0], k_shield=s.k, shield_scale=SHIELD_SCALE, cond_max=COND_MAX,
                           max_attempts=MAX_ATTEMPTS, batch_id=1, U=s.U, Y=s.Y)
    elif call == "static":
        g.gelo_qkv_forward_static(s.ctx, s.kind, s.H[0], s.W[0], s.Z[0], s.U, s.Y, k_shield=s.k, shield_scale=SHIELD_SCALE, batch_id=1)
    elif call == "ahead":
        mixings = g.gelo_sample_mixing_batch(s.ctx, s.kind, s.case["n_data"], s.k, s.case["d"], s.code, 1, s.case["layers"])
        for H, W, Z, m in zip(s.H, s.W, s.Z, mixings):
            g.gelo_chain(s.ctx, m, H, W, Z, s.U, s.Y, shield_scale=SHIELD_SCALE)
            g.gelo_mixing_free(s.ctx, m)
    else:
        g.gelo_mix(s.ctx, s.mixing, s.H[0], s.U, shield_scale=SHIELD_SCALE)
        g.gelo_project_fp8(s.ctx, s.U, s.Wq, s.case["p"], s.Y)
        g.gelo_unmix(s.ctx, s.mixing, s.Y, s.Z[0])
    # U and Y are the messages the accelerator sees (of the last layer, where layers share the buffers), Z the results
    return {"Z": s.Z, "U": s.U, "Y": s.Y}


def _block_sizes(n, block=256):
    return [min(block, n - r) for r in range(0, n, block)]


def work(case):
    n_data, k, d, p, layers = (case[x] for x in ("n_data", "k_shield", "d", "p", "layers"))
    kind, n = case["kind"], n_data + k
    size = 2 if case["dtype"] == "bf16" else 4
    weight = d * p * (1 if case["call"] == "fp8" else size)
    # hidden states and weight in; U, Y and Z out, and U and Y in again on the other side of the protocol
    moved = (n_data * d + n_data * p + 2 * n * d + 2 * n * p) * size + weight
    project = 2 * n * d * p
    if kind == "structured":
        # three rounds of a Walsh-Hadamard transform over the row blocks of n's binary expansion, additions only
        adds = 3 * sum((1 << b) * b for b in range(n.bit_length()) if n >> b & 1)
        mixing, drawn = adds * (d + p), 0
    elif kind == "blocks":
        sizes = _block_sizes(n)
        mixing = sum(2 * b * b * d for b in sizes) + round(sum(2 * b * b * p for b in sizes) * n_data / n)
        drawn = sum(8 * b ** 3 // 3 for b in sizes)
    else:
        mixing = 2 * n * n * d + 2 * n_data * n * p
        # QR with explicit Q; the product of reflectors alone; LU with inverse (one attempt); both
        drawn = {"orthogonal": 8 * n ** 3 // 3, "reflectors": 4 * n ** 3 // 3, "gaussian": 2 * n ** 3,
                 "conditioned": 8 * n ** 3 // 3 + 2 * n ** 3}[kind]
    if case["call"] == "fp8":
        drawn = 0
    return {"bytes": layers * moved, "flops": layers * (project + mixing + drawn)}


def tolerance(case):
    """About four times the distance of this path's outputs from the same path in 64 bits, taken over kinds, sizes and seeds."""
    n = case["n_data"] + case["k_shield"]
    if case["call"] == "fp8":
        # U rounded another way moves 8-bit codes (a step of 2^-3 each), which the unmix passes on: 0.013 in Y and 0.031 in Z
        # where half of U's values moved by one rounding
        return {"rel": 2e-2, "max": 0.5}
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.4}          # roundings of A, U, Y and Z: 0.003 in U and Y, 0.004 to 0.009 in Z
    if case["kind"] == "gaussian":
        return {"rel": 6e-4, "max": 2e-2}         # Z carries kappa(A) <= 1e3: 0.3e-4 to 1.4e-4
    if case["kind"] in ("structured", "reflectors"):
        return {"rel": 1e-5, "max": 1e-4}         # 0.3e-6 to 2.6e-6
    # the QR factor moves by the rounding error times the condition number of its n x n Gaussian, which grows like n with a heavy
    # tail: 4e-7 (18 rows), 5e-6 (543), 1e-5 and 7.6e-5 (2150, two seeds); conditioned, Z: 7.5e-5 (1575 rows)
    n = min(n, 256) if case["kind"] == "blocks" else n
    rel = max(1e-5, 1.5e-7 * n)
    return {"rel": rel, "max": 30 * rel}
