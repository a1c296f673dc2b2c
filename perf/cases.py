"""The attention forward pass as a user's program calls it: what is timed, on which inputs, and how exact it has to be.

Every case is one call of ``fa2_fwd`` on torch tensors, outputs allocated by the call unless the case says that the
program keeps them.  Sizes are those of the repository's own workloads, of the paper's benchmark and of its tests, or
generic ones for the uses between them (a prompt of odd length, a chunk of queries, a decoding step).
"""
import math

import torch

import paper_2312_11918_amd as fa2

DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16}


def _case(name, B, H, Nq, Nk, d, dtype, causal=False, lse=True, outliers=0.0, keep=False):
    return {"name": name, "B": B, "H": H, "Nq": Nq, "Nk": Nk, "d": d, "dtype": dtype, "causal": causal, "lse": lse,
            "outliers": outliers, "keep": keep}


def listed():
    return [
        # The smallest workload: one short sequence, two heads.  Latency of the call and of one launch.
        _case("tiny_N256_d64", 1, 2, 256, 256, 64, "fp16"),
        # Many short sequences: a batch of sentences through an encoder.
        _case("short_N512_d64", 32, 16, 512, 512, 64, "fp16"),
        # The headline: 16k tokens in sequences of ordinary length, forward pass of a training step.  The program
        # keeps its output buffers.
        _case("train_N2048_d128", 8, 16, 2048, 2048, 128, "fp16", keep=True),
        # The same tokens with the decoder's mask, in bfloat16.
        _case("causal_N2048_d128_bf16", 8, 16, 2048, 2048, 128, "bf16", causal=True),
        # A batch whose sequences were cut to one token less (next-token targets): no size is a whole tile.
        _case("ragged_N2047_d128", 8, 16, 2047, 2047, 128, "fp16"),
        # Long sequences, where streaming K and V decides.
        _case("long_N8192_d128_bf16", 2, 16, 8192, 8192, 128, "bf16"),
        # The longest workload, with one per cent of large keys (outlier tokens).
        _case("longest_N16384_d64_outliers", 1, 32, 16384, 16384, 64, "fp16", outliers=0.01),
        # The paper's benchmark shape with the largest head dimension.
        _case("paper_N4096_d256", 4, 8, 4096, 4096, 256, "fp16"),
        # One prompt of odd length under the decoder's mask: prefill for a single user.
        _case("prompt_N1111_d128_bf16", 1, 16, 1111, 1111, 128, "bf16", causal=True, lse=False),
        # A chunk of queries against one slice of a long key range; its LSE is needed to merge the slices.
        _case("chunk_Nq512_Nk8192_d128_bf16", 1, 16, 512, 8192, 128, "bf16"),
        # One decoding step of a batch: one new query per sequence against its cached keys.
        _case("decode_B16_Nk2048_d128_bf16", 16, 16, 1, 2048, 128, "bf16", lse=False),
        # One decoding step of a single long sequence whose length is no round number.
        _case("decode_B1_Nk16001_d64", 1, 32, 1, 16001, 64, "fp16", lse=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# no drawn case costs more than the largest listed ones (the longest workload's arithmetic, its and the headline's bytes)
MAX_FLOPS = 4.0 * 32 * 16384.0 ** 2 * 64
MAX_BYTES = 270e6


def draw(rng):
    while True:
        use = rng.choice(("self", "self", "causal", "causal", "chunk", "decode", "decode"))
        d = rng.choice((64, 64, 128, 128, 128, 256))
        H = rng.choice((2, 6, 8, 12, 16, 24, 32))
        if use == "chunk":
            Nq, Nk = _log_int(rng, 2, 2048), _log_int(rng, 64, 16384)
            B = _log_int(rng, 1, 16)
        elif use == "decode":
            Nq, Nk = 1, _log_int(rng, 64, 32768)
            B = _log_int(rng, 1, 64)
        else:
            Nq = _log_int(rng, 64, 16384)
            if rng.random() < 0.5:   # a padded length: whole tiles
                Nq = max(128, (Nq + 64) // 128 * 128)
            Nk = Nq
            B = _log_int(rng, 1, 64)
        case = {"B": B, "H": H, "Nq": Nq, "Nk": Nk, "d": d, "dtype": rng.choice(("fp16", "bf16")),
                "causal": use == "causal", "lse": use == "chunk" or rng.random() < 0.5,
                "outliers": 0.01 if use == "self" and rng.random() < 0.2 else 0.0, "keep": rng.random() < 0.2}
        w = work(case)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return case


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, H, Nq, Nk, d = (case[x] for x in ("B", "H", "Nq", "Nk", "d"))

    def normal(n):
        return torch.randn((B, n, H, d), generator=g, device="cuda")

    q, k, v = normal(Nq), normal(Nk), normal(Nk)
    if case["outliers"]:
        large = torch.rand((B, Nk, H, 1), generator=g, device="cuda") < case["outliers"]
        k = torch.where(large, 8.0 * k, k)
    dtype = DTYPES[case["dtype"]]
    state = {"q": q.to(dtype), "k": k.to(dtype), "v": v.to(dtype), "scale": d ** -0.5, "causal": case["causal"],
             "return_lse": case["lse"], "out": None, "lse": None}
    if case["keep"]:
        state["out"] = torch.empty_like(state["q"])
        if case["lse"]:
            state["lse"] = torch.empty((B, H, Nq), dtype=torch.float32, device="cuda")
    return state


def run(state):
    return fa2.fa2_fwd(state["q"], state["k"], state["v"], state["scale"], out=state["out"], lse=state["lse"],
                       return_lse=state["return_lse"], causal=state["causal"])


def work(case):
    B, H, Nq, Nk, d = (case[x] for x in ("B", "H", "Nq", "Nk", "d"))
    # query-key pairs that count: under the mask the diagonal and what lies below it
    pairs = Nq * (Nq + 1) / 2.0 if case["causal"] else float(Nq) * Nk
    values = 2.0 * B * H * d * (2 * Nq + 2 * Nk)   # Q, K, V read once and O written once, 16 bits each
    return {"bytes": values + (4.0 * B * H * Nq if case["lse"] else 0.0), "flops": 4.0 * B * H * pairs * d}


def tolerance(case):
    # Rounding P and O to 16 bits: against the same formula in 64 bits O is off by 2.4e-4...2.9e-4 in fp16 and by
    # 2.0e-3...2.4e-3 in bf16 (2-norm, over all listed cases), its worst element by 1.3e-3 and 2.2e-2 of the larger of
    # itself and the root mean square; the fp32 LSE by under 1e-7.  Four times that.
    return {"rel": 1.2e-3, "max": 6e-3} if case["dtype"] == "fp16" else {"rel": 1e-2, "max": 9e-2}


def exact(case, seed):
    # The formula head by head in 64 bits, a block of queries at a time, on the inputs that prepare() makes.  The
    # longest workload takes under 5 seconds.
    state = prepare(case, seed)
    B, H, Nq, Nk, d = (case[x] for x in ("B", "H", "Nq", "Nk", "d"))
    o = torch.empty((B, Nq, H, d), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, H, Nq), dtype=torch.float64, device="cuda")
    keys = torch.arange(Nk, device="cuda")
    block = 4096
    for b in range(B):
        for h in range(H):
            q, k, v = (state[x][b, :, h].double() for x in ("q", "k", "v"))
            kt = k.t().contiguous()
            for i in range(0, Nq, block):
                s = q[i:i + block] @ kt * state["scale"]
                if case["causal"]:
                    s.masked_fill_(keys[None, :] > torch.arange(i, i + s.shape[0], device="cuda")[:, None], -math.inf)
                total = torch.logsumexp(s, 1)
                lse[b, h, i:i + block] = total
                o[b, i:i + block, h] = s.sub_(total[:, None]).exp_() @ v
    return o, lse if case["lse"] else None
