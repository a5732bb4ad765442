"""The attention calls whose speed this library is judged by.

A case is one pass of attention through the public entry points of
`paper_2505_14201_amd.flashd`: `attn_fwd` (prefill and decode), `attn_fwd_kv8` (K and V
stored as fp8) or a run of `attn_fwd_state` calls (keys arriving in chunks).  Tensors are
allocated once, as a serving loop or a training step would have them, and the outputs are
the caller's own buffers.

Fields of a case: op ("attn", "kv8" or "chunks"), dtype of Q and O, B, Hq, Hkv, Lq, Lk, d,
causal, chunks (how many equal runs the keys arrive in), std (standard deviation of Q and K),
plant (share of query rows with a dominant key), sink (one dominant early key per kv head).
"""
import math

import torch

from paper_2505_14201_amd import flashd

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
FP8_SCALE = 2.0 ** -5       # of N(0, 1) values: 32 sigma-units per 1.0, +-14 sigma fit e4m3


def _case(name, op="attn", dtype="bf16", B=1, Hq=32, Hkv=32, Lq=1, Lk=1, d=128, causal=False,
          chunks=1, std=1.0, plant=0.0, sink=0.0):
    c = {"op": op, "dtype": dtype, "B": B, "Hq": Hq, "Hkv": Hkv, "Lq": Lq, "Lk": Lk, "d": d,
         "causal": causal, "chunks": chunks, "std": std, "plant": plant, "sink": sink}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: one fp32 head of 128 positions (a unit test, a probe of a single
        # layer); launch latency and the host path count.
        _case("single_head_f32", dtype="f32", Hq=1, Hkv=1, Lq=128, Lk=128, d=64),
        # fp32 reference runs of a small model: a batch of ragged causal sequences.
        _case("causal_ragged_f32", dtype="f32", B=2, Hq=12, Hkv=12, Lq=777, Lk=777, d=64,
              causal=True),
        # A prompt of ordinary, ragged length in a grouped-query model, few sequences at a time.
        _case("prompt_ragged_gqa_bf16", B=2, Hq=32, Hkv=8, Lq=1000, Lk=1000, causal=True),
        # The batch prefill of a 7B-sized model.
        _case("causal_prefill_bf16", B=4, Lq=2048, Lk=2048, causal=True),
        # One long document without a mask: the largest call.
        _case("long_noncausal_bf16", Lq=16384, Lk=16384),
        # fp16 with heads of 64 and scores of several hundred, dominant keys planted.
        _case("wide_scores_causal_f16", dtype="f16", B=2, Hq=16, Hkv=16, Lq=4096, Lk=4096, d=64,
              causal=True, std=4.0, plant=0.05),
        # Prefill whose keys arrive in two chunks, the state handed from one call to the next.
        _case("two_chunks_bf16", op="chunks", B=4, Lq=2048, Lk=2048, causal=True, chunks=2),
        # One user's token in a short context: latency of a single decode step.
        _case("decode_one_short_bf16", Hq=32, Hkv=8, Lk=1000),
        # The batched decode step of a serving loop.
        _case("decode_batch_bf16", B=64, Hq=32, Hkv=8, Lk=8192),
        # One sequence with a context of 128 K: the keys are split over the whole chip.
        _case("decode_one_long_bf16", Hq=32, Hkv=8, Lk=131072),
        # The batched decode step on a KV cache kept in fp8.
        _case("decode_batch_fp8_kv", op="kv8", B=64, Hq=32, Hkv=8, Lk=8192),
        # 16 positions per sequence at once: drafted tokens being checked, a short prompt chunk.
        _case("decode_16_positions_bf16", B=64, Hq=32, Hkv=8, Lq=16, Lk=8192, causal=True),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread evenly over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


HEADS = [(32, 8), (32, 32), (16, 16), (32, 4), (12, 12), (8, 1), (16, 2), (8, 8)]


def _bounded(c, flops=1.0e12, size=1.2e9):
    """The case with its batch cut until it stays below the given work."""
    w = work(c)
    over = max(w["flops"] / flops, w["bytes"] / size, 1.0)
    return dict(c, B=max(1, int(c["B"] / over)))


def draw(rng):
    kind = rng.choices(["prefill", "decode", "kv8", "chunks", "f32"], [35, 30, 13, 10, 12])[0]
    hq, hkv = rng.choice(HEADS)
    d = rng.choice([64, 128, 128])
    dtype = rng.choice(["bf16", "bf16", "f16"])
    causal = rng.random() < 0.7
    if kind == "f32":
        # fp32: tests, probes and reference runs of small models
        lk = _log(rng, 16, 2048)
        lq = lk if rng.random() < 0.75 else _log(rng, 1, lk)
        h = rng.choice([1, 4, 8, 12, 16])
        return _bounded(_case("", dtype="f32", B=_log(rng, 1, 8), Hq=h, Hkv=h, Lq=lq, Lk=lk,
                              d=rng.choice([64, 64, 128]), causal=causal), flops=6.0e9)
    if kind in ("prefill", "chunks"):
        lk = _log(rng, 16 if kind == "prefill" else 256, 12288)
        if rng.random() < 0.4:
            lk = max(64, lk // 64 * 64)
        # mostly whole prompts, otherwise queries late in a context
        lq = lk if rng.random() < 0.75 else _log(rng, max(1, lk // 16), lk)
        chunks = rng.randint(2, 4) if kind == "chunks" else 1
        lk = lk // chunks * chunks
        lq = min(lq, lk)
        wide = hq == hkv and kind == "prefill" and rng.random() < 0.25
        return _bounded(_case("", op="attn" if kind == "prefill" else "chunks", dtype=dtype,
                              B=_log(rng, 1, 64), Hq=hq, Hkv=hkv, Lq=lq, Lk=lk, d=d, causal=causal,
                              chunks=chunks, std=4.0 if wide else 1.0, plant=0.05 if wide else 0.0),
                        size=6.0e8)
    # decode steps, with the cache in the storage type of Q or in fp8; a fifth with several
    # positions per sequence, and for fp8 now and then a whole prompt
    lk = _log(rng, 32, 131072)
    lq = 1 if rng.random() < 0.75 else _log(rng, 2, 16)
    if kind == "kv8" and rng.random() < 0.3:
        lk = _log(rng, 128, 4096)
        lq = lk
    sink = 8.0 if kind == "decode" and lk >= 256 and rng.random() < 0.15 else 0.0
    return _bounded(_case("", op="attn" if kind == "decode" else "kv8", dtype=dtype,
                          B=_log(rng, 1, 64), Hq=hq, Hkv=hkv, Lq=min(lq, lk), Lk=lk, d=d,
                          causal=lq > 1, std=4.0 if sink else 1.0, sink=sink))


def _plant(gen, q, k, share, causal):
    """For a share of the query rows i, a key j visible to i becomes 8 q_i (the last such row
    wins where two pick the same key)."""
    B, H, Lq, d = q.shape
    Lk = k.shape[2]
    rows = torch.arange(Lq, device=q.device).expand(B, H, Lq)
    seen = (rows + (Lk - Lq) + 1).clamp(0, Lk) if causal else torch.full_like(rows, Lk)
    pick = torch.rand(B, H, Lq, device=q.device, generator=gen) < share
    j = (torch.rand(B, H, Lq, device=q.device, generator=gen) * seen).long().clamp(max=Lk - 1)
    src = torch.where(pick & (seen > 0), rows, torch.full_like(rows, -1))
    owner = torch.full((B, H, Lk), -1, dtype=torch.long, device=q.device)
    owner.scatter_reduce_(2, j, src, "amax")
    idx = owner.clamp(min=0).unsqueeze(-1).expand(B, H, Lk, d)
    big = (q.float() * 8.0).to(k.dtype)
    return torch.where((owner >= 0).unsqueeze(-1), torch.gather(big, 2, idx), k).contiguous()


def _sinks(gen, q, k, gain):
    """Per kv head one early key along the sum of its group's last queries."""
    B, Hq, Lq, d = q.shape
    Hkv, Lk = k.shape[1], k.shape[2]
    g = Hq // Hkv
    pos = (torch.rand(B, Hkv, device=q.device, generator=gen) * max(1, Lk // 64)).long()
    key = q[:, :, Lq - 1].float().view(B, Hkv, g, d).sum(2) * (gain / g)
    k.scatter_(2, pos.view(B, Hkv, 1, 1).expand(B, Hkv, 1, d), key.to(k.dtype).unsqueeze(2))
    return k


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = DTYPES[c["dtype"]]

    def normal(H, L, std):
        x = torch.randn(c["B"], H, L, c["d"], device="cuda", dtype=dt, generator=gen)
        return x.mul_(std) if std != 1.0 else x

    q = normal(c["Hq"], c["Lq"], c["std"])
    k = normal(c["Hkv"], c["Lk"], c["std"])
    v = normal(c["Hkv"], c["Lk"], 1.0)
    if c["plant"] > 0.0:
        k = _plant(gen, q, k, c["plant"], c["causal"])
    if c["sink"] > 0.0:
        k = _sinks(gen, q, k, c["sink"])
    s = {"case": c, "q": q, "o": torch.empty_like(q), "scale": 1.0 / math.sqrt(c["d"])}
    if c["op"] == "kv8":
        s["k"] = (k / FP8_SCALE).to(torch.float8_e4m3fn)
        s["v"] = (v / FP8_SCALE).to(torch.float8_e4m3fn)
    elif c["op"] == "chunks":
        n = c["Lk"] // c["chunks"]
        s["parts"] = [(k[:, :, i * n:(i + 1) * n].contiguous(), v[:, :, i * n:(i + 1) * n].contiguous(),
                       c["Lk"] - c["Lq"] - i * n) for i in range(c["chunks"])]
        s["state"] = torch.empty(c["B"], c["Hq"], c["Lq"], c["d"] + 2, dtype=torch.float32,
                                 device="cuda")
    else:
        s["k"], s["v"] = k, v
    return s


def run(state):
    s = state
    c = s["case"]
    if c["op"] == "kv8":
        flashd.attn_fwd_kv8(s["q"], s["k"], s["v"], s["o"], c["causal"], s["scale"], FP8_SCALE,
                            FP8_SCALE)
        return s["o"]
    if c["op"] == "chunks":
        st = s["state"]
        last = len(s["parts"]) - 1
        for i, (k, v, shift) in enumerate(s["parts"]):
            # the last call hands out the output and the state that further keys would join
            flashd.attn_fwd_state(s["q"], k, v, c["causal"], s["scale"],
                                  o=s["o"] if i == last else None,
                                  state_in=st if i > 0 else None, state_out=st, causal_shift=shift)
        return s["o"], st
    flashd.attn_fwd(s["q"], s["k"], s["v"], s["o"], c["causal"], s["scale"])
    return s["o"]


def work(case):
    c = case
    lq, lk = c["Lq"], c["Lk"]
    if c["causal"]:
        off = lk - lq                       # row i sees i + off + 1 keys, off >= 0
        pairs = lq * (off + 1) + lq * (lq - 1) // 2
    else:
        pairs = lq * lk
    size = 4 if c["dtype"] == "f32" else 2
    nq = c["B"] * c["Hq"] * lq * c["d"]
    nk = c["B"] * c["Hkv"] * lk * c["d"]
    moved = 2 * nq * size + 2 * nk * (1 if c["op"] == "kv8" else size)
    if c["op"] == "chunks":
        moved += c["B"] * c["Hq"] * lq * (c["d"] + 2) * 4      # the state that is handed out
    return {"bytes": moved, "flops": 4 * c["d"] * c["B"] * c["Hq"] * pairs}


def tolerance(case):
    # Against attention in fp64 on the same inputs the worst of the listed and of 24 drawn cases
    # is 1.6e-7 (f32), 3.2e-4 (f16) and 2.5e-3 (bf16): the last two are the rounding of the
    # weights and of the output to the storage type.  Four to six times that.
    return {"rel": {"f32": 1e-6, "f16": 1.3e-3, "bf16": 1e-2}[case["dtype"]]}
