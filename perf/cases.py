"""The work this library is timed on: calls of its public entry points over the range of sizes they serve.

A case is one call (``run``) on inputs that live on the GPU (``prepare``).  Decode calls (up to 128 activation
rows, attention, grouped layers) go through the marshalled handle that ``prepare=True`` returns, as a serving loop
with static buffers makes them; calls of more rows go through the plain function with a fresh output tensor, as a
prompt of another length every time makes them.  Sizes are those of the benchmark (bench.py, bench_extras.py), and
odd ones between them.
"""
import math

import torch

from paper_2605_13915_amd import binding as msd

_OUT = {"f32": torch.float32, "bf16": torch.bfloat16}


# ------------------------------------------------------------------ cases
def listed():
    return [
        # one token of one user through a square projection: the smallest call, launch latency and 17 MB of weights
        dict(name="w8_one_row", kind="w8", M=1, K=4096, N=4096, packed=True, out="f32"),
        # a small decode batch through the wide projection of a block
        dict(name="w8_decode_8", kind="w8", M=8, K=4096, N=14336, packed=True, out="bf16"),
        # a large, odd decode batch on weights as the checkpoint has them
        dict(name="w8_decode_100", kind="w8", M=100, K=4096, N=4096, packed=False, out="bf16"),
        # the rest of a prompt (chunked prefill): an odd number of rows between decode and prefill
        dict(name="w8_chunk_777", kind="w8", M=777, K=4096, N=14336, packed=True, out="bf16"),
        # a full prefill batch of the largest layer
        dict(name="w8_prefill", kind="w8", M=2048, K=8192, N=28672, packed=True, out="f32"),
        # the 4-bit layer: one token, a decode batch on unpacked weights, prefill
        dict(name="w4_one_row", kind="w4", M=1, K=8192, N=28672, packed=True, out="f32"),
        dict(name="w4_decode_32", kind="w4", M=32, K=8192, N=28672, packed=False, out="f32"),
        dict(name="w4_prefill", kind="w4", M=4096, K=8192, N=28672, packed=True, out="bf16"),
        # grouped-query attention, one decode step: a batch of users with contexts of different lengths, and a batch
        # of long contexts with the scales per channel
        dict(name="attn_ragged_4k", kind="attn", B=16, Hq=32, Hkv=8, L=4096, mode="token", ragged=True, out="f32"),
        dict(name="attn_32k", kind="attn", B=16, Hq=32, Hkv=8, L=32768, mode="channel", ragged=False, out="bf16"),
        # attention over a latent cache, every head of a large model
        dict(name="mla_128_heads", kind="mla", B=32, Hq=128, L=4096, mode="token", ragged=False, out="f32"),
        # an expert layer: the rows of a decode batch spread over the experts
        dict(name="moe_w8_64", kind="moe8", T=64, E=64, K=4096, N=2048, out="f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choice(["w8", "w8", "w8", "w4", "w4", "attn", "attn", "mla", "moe8", "moe4"])
    out = rng.choice(["f32", "bf16"])
    if kind in ("w8", "w4"):
        # half of the calls are decode batches, half are longer; K and N of layers from 1024 to 28672 wide, most
        # of them round, the rest any width the format takes
        M = _log(rng, 1, 128) if rng.random() < 0.5 else _log(rng, 129, 8192)
        unit = 64 if kind == "w8" else 512
        if rng.random() < 0.15:
            unit = 16 if kind == "w8" else 32
        K = max(1, _log(rng, 1024, 14336) // unit) * unit
        N = _log(rng, 512, 28672)
        if rng.random() < 0.8:
            N = N // 128 * 128
        packed = rng.random() < 0.6 and K % (64 if kind == "w8" else 512) == 0
        return dict(kind=kind, M=M, K=K, N=N, packed=packed, out=out)
    mode = rng.choice(["token", "channel"])
    ragged = rng.random() < 0.5
    if kind == "attn":
        Hkv = rng.choice([1, 2, 4, 8])
        return dict(kind=kind, B=_log(rng, 1, 64), Hq=Hkv * rng.choice([1, 2, 4, 4, 6, 8, 12, 16]), Hkv=Hkv,
                    L=_log(rng, 64, 32768), mode=mode, ragged=ragged, out=out)
    if kind == "mla":
        return dict(kind=kind, B=_log(rng, 1, 64), Hq=rng.choice([8, 16, 32, 40, 64, 128]), L=_log(rng, 64, 32768),
                    mode=mode, ragged=ragged, out=out)
    unit = 64 if kind == "moe8" else 128
    return dict(kind=kind, T=_log(rng, 1, 1024), E=rng.choice([8, 16, 32, 64, 128]),
                K=max(1, _log(rng, 1024, 7168) // unit) * unit, N=_log(rng, 512, 4096) // 64 * 64, out=out)


def draw(rng):
    """One more case; no larger than the largest listed one, and its buffers no larger than the largest listed ones."""
    top = [work(c) for c in listed()]
    most_bytes, most_flops = max(w["bytes"] for w in top), max(w["flops"] for w in top)
    while True:
        c = _draw_once(rng)
        w = work(c)
        if max(w["bytes"], _held(c)) <= most_bytes and w["flops"] <= most_flops:
            return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _activations(g, M, K):
    """BF16 N(0,1) rows, 1 % of the channels fifty times larger (the outlier channels of real activations)."""
    x = torch.randn((M, K), device="cuda", generator=g)
    idx = torch.randperm(K, device="cuda", generator=g)[: max(1, K // 100)]
    x[:, idx] *= 50.0
    return x.to(torch.bfloat16)


def _int8_weights(g, *shape):
    W = torch.empty(shape, dtype=torch.int8, device="cuda").random_(-127, 128, generator=g)
    s = torch.rand(shape[:-1], device="cuda", generator=g) * 0.009 + 0.001
    return W, s


def _mxfp4_weights(g, *shape):
    """N(0, 0.02) weights quantised to OCP MXFP4: E2M1 nibbles [..., K/2] and E8M0 bytes [..., K/32]."""
    K = shape[-1]
    rows = math.prod(shape[:-1])
    codes = torch.empty((rows, K // 2), dtype=torch.uint8, device="cuda")
    exps = torch.empty((rows, K // 32), dtype=torch.uint8, device="cuda")
    edges = torch.tensor([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0], device="cuda")
    step = max(1, (1 << 26) // K)
    for r in range(0, rows, step):
        n = min(step, rows - r)
        w = (torch.randn((n, K // 32, 32), device="cuda", generator=g) * 0.02)
        _, e = torch.frexp(w.abs().amax(dim=2).clamp_min(1e-30))  # max = f * 2^e, f in [0.5, 1)
        e = e - 1 - 2                                               # the largest binade of E2M1 is 2^2
        w = torch.ldexp(w, -e[:, :, None])
        nib = torch.bucketize(w.abs(), edges).to(torch.uint8)
        nib |= (w < 0).to(torch.uint8) << 3
        nib = nib.view(n, K // 2, 2)
        codes[r:r + n] = nib[:, :, 0] | (nib[:, :, 1] << 4)
        exps[r:r + n] = (e + 127).to(torch.uint8)
    return codes.view(*shape[:-1], K // 2), exps.view(*shape[:-1], K // 32)


def _cache_rows(g, shape, mode):
    """INT8 cache [..., L][channels] of N(0,1) values: scales per token (row maximum) or per channel."""
    n, ch = math.prod(shape[:-1]), shape[-1]
    codes = torch.empty((n, ch), dtype=torch.int8, device="cuda")
    scale = torch.empty((n,), device="cuda") if mode == "token" else None
    step = max(1, (1 << 27) // ch)
    for r in range(0, n, step):
        x = torch.randn((min(step, n - r), ch), device="cuda", generator=g)
        if mode == "token":
            s = x.abs().amax(dim=1, keepdim=True) / 127.0
            scale[r:r + step] = s[:, 0]
            x /= s
        else:
            x *= 127.0 / 5.5  # the largest of the values of a channel lies at 5.5 or so; the few beyond saturate
        codes[r:r + step] = x.round_().clamp_(-127, 127).to(torch.int8)
    return codes.view(shape), scale


def _lengths(g, B, L, ragged):
    return torch.randint((L + 1) // 2, L + 1, (B,), dtype=torch.int32, device="cuda", generator=g) if ragged else None


def prepare(case, seed):
    g = _gen(seed)
    kind, out = case["kind"], _OUT[case["out"]]
    if kind in ("w8", "w4"):
        M, K, N = case["M"], case["K"], case["N"]
        x = _activations(g, M, K)
        if kind == "w8":
            W, s = _int8_weights(g, N, K)
            fn, weights = (msd.msd_gemm_w8a16_packed, (msd.msd_pack_weights_w8(W), s)) if case["packed"] else (msd.msd_gemm_w8a16, (W, s))
        else:
            W, e = _mxfp4_weights(g, N, K)
            fn, weights = (msd.msd_gemm_w4a16_packed, (*msd.msd_pack_weights_w4(W, e), N)) if case["packed"] else (msd.msd_gemm_w4a16, (W, e))
        if M <= 128:
            return fn(x, *weights, out_dtype=out, prepare=True)
        return lambda: fn(x, *weights, out_dtype=out)
    if kind in ("moe8", "moe4"):
        T, E, K, N = case["T"], case["E"], case["K"], case["N"]
        x = _activations(g, T, K)
        counts = torch.bincount(torch.randint(0, E, (T,), device="cuda", generator=g), minlength=E)
        offs = torch.zeros(E + 1, dtype=torch.int32, device="cuda")
        offs[1:] = torch.cumsum(counts, 0)
        if kind == "moe8":
            return msd.msd_moe_gemm_w8a16(x, offs, *_int8_weights(g, E, N, K), out_dtype=out, prepare=True)
        return msd.msd_moe_gemm_w4a16(x, offs, *_mxfp4_weights(g, E, N, K), out_dtype=out, prepare=True)
    B, Hq, L, mode = case["B"], case["Hq"], case["L"], case["mode"]
    scale_mode = msd.MSD_PER_TOKEN if mode == "token" else msd.MSD_PER_CHANNEL
    n = _lengths(g, B, L, case["ragged"])
    if kind == "attn":
        Hkv, d = case["Hkv"], 128
        q = torch.randn((B, Hq, d), device="cuda", generator=g).to(torch.bfloat16)
        Kc, ks = _cache_rows(g, (B, Hkv, L, d), mode)
        Vc, vs = _cache_rows(g, (B, Hkv, L, d), mode)
        if mode == "token":
            ks, vs = ks.view(B, Hkv, L), vs.view(B, Hkv, L)
        else:
            ks, vs = (torch.rand((Hkv, d), device="cuda", generator=g) * 0.02 + 0.03 for _ in range(2))
        return msd.msd_attn_decode_int8kv(q, Kc, Vc, ks, vs, scale_mode, kv_len=n, out_dtype=out, prepare=True)
    q = torch.randn((B, Hq, 576), device="cuda", generator=g).to(torch.bfloat16)
    C, cs = _cache_rows(g, (B, L, 576), mode)
    cs = cs.view(B, L) if mode == "token" else torch.rand(576, device="cuda", generator=g) * 0.02 + 0.03
    # (128 + 64)^-0.5: the softmax scale of a head of 128 channels and 64 positional ones
    return msd.msd_mla_decode_int8kv(q, C, cs, scale_mode, 192 ** -0.5, kv_len=n, out_dtype=out, prepare=True)


def run(state):
    return state()


# ------------------------------------------------------------------ what a pass cannot do without
def _held(case):
    """Bytes of the weights or cache that the case keeps on the GPU."""
    k = case["kind"]
    if k == "moe8":
        return case["E"] * case["K"] * case["N"]
    if k == "moe4":
        return case["E"] * case["K"] * case["N"] * 17 // 32
    if k == "attn":
        return 2 * case["B"] * case["Hkv"] * case["L"] * 128
    if k == "mla":
        return case["B"] * case["L"] * 576
    return case["K"] * case["N"]


def work(case):
    """Each input read once, each output written once; the multiplications and additions of the two products of
    every weight (or cached value) with the two components of an activation."""
    k, ob = case["kind"], 4 if case["out"] == "f32" else 2
    if k in ("w8", "w4", "moe8", "moe4"):
        M, K, N = case.get("M", case.get("T")), case["K"], case["N"]
        # experts that the rows of a batch reach
        e = case["E"] * (1.0 - (1.0 - 1.0 / case["E"]) ** M) if "E" in case else 1.0
        w = K * N + 4 * N if k in ("w8", "moe8") else K * N * 17 / 32
        return {"bytes": e * w + 2.0 * M * K + ob * M * N, "flops": 4.0 * M * K * N}
    B, Hq = case["B"], case["Hq"]
    toks = B * case["L"] * (0.75 if case["ragged"] else 1.0)
    if k == "attn":
        by = toks * case["Hkv"] * (256 + (8 if case["mode"] == "token" else 0)) + B * Hq * 128 * (2 + ob)
        return {"bytes": by, "flops": 4.0 * toks * Hq * 256}
    by = toks * (576 + (4 if case["mode"] == "token" else 0)) + B * Hq * (2 * 576 + ob * 512)
    return {"bytes": by, "flops": 4.0 * toks * Hq * 1088}


def tolerance(case):
    k = case["kind"]
    if case["out"] == "bf16":
        return {"rel": 4e-3}  # one rounding to BF16: 1.7e-3 from the same path with its output in 64 bits
    if k in ("w8", "moe8"):
        return {"rel": 1.5e-7}  # exact integer sums, then four fp32 roundings: 3.6e-8 from the merge in 64 bits
    if k in ("w4", "moe4"):
        return {"rel": 1e-6}  # fp32 sums of block products, exact or a few roundings away in any order
    # the softmax numerators are decomposed relative to a bound that depends on the tile of tokens: 4e-5 to 9e-5 from
    # the attention in 64 bits, whatever the tile
    return {"rel": 3.5e-4}
