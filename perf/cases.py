"""The decode-attention calls a program makes through this package, as cases
that can be timed and checked.

Each case is one `entry` with its sizes:

  decode     da_decode_attn over a dense [B, L, H_KV, 128] cache (planned inside the call)
  noalloc    da_decode_attn_noalloc over the same layout, into a preallocated output
  varlen     da_decode_attn with cu_seqlens_k: a batch of mixed lengths, packed
  paged      da_decode_attn_paged: the same in a paged cache, lengths on the device
  scheduled  da_decode_attn_scheduled: per-sequence split counts planned from host-known lengths,
             kept by the caller beside the cache (packed when page is 0, else paged)
  partials   da_split_partials then da_combine_splits: chunk states as a context-parallel
             rank hands them on, and their merge
  step       a captured HIP graph of one call per layer with plans for K/V streamed from HBM:
             a decode step as a serving loop replays it

Lengths of a mixed batch follow from the case alone (`lens`, `len_lo`,
`len_hi`, `len_seed`), so its work is known; the seed of prepare() draws the
tensors.  Queries have twice unit variance's deviation, so that the softmax
has the sharp and flat rows real scores have.
"""

import math

import numpy as np
import torch

import paper_2604_00028_amd as da

D = 128
DEV = "cuda"
# (query heads, KV heads): MQA, GQA groups of 4 to 64, and no sharing
HEADS = [(8, 1), (32, 1), (16, 2), (32, 2), (128, 2), (32, 4), (64, 4), (64, 8), (40, 8), (128, 16), (16, 16)]
MAX_KV_BYTES = 1 << 30


def listed():
    return [
        # the smallest call: one MQA sequence of 128 keys, bound by launch and latency
        {"name": "mqa_b1_l128", "entry": "decode", "B": 1, "H_Q": 8, "H_KV": 1, "L": 128},
        # low-tile pure MQA, a few short sequences of odd length
        {"name": "mqa32_b4_l507", "entry": "decode", "B": 4, "H_Q": 32, "H_KV": 1, "L": 507},
        # Llama-3.1-70B decode heads at batch 1: all 80 layers of a step in one graph, caches read from HBM
        {"name": "step_gqa_b1_l512_x80", "entry": "step", "B": 1, "H_Q": 64, "H_KV": 8, "L": 512, "layers": 80},
        # the same heads, one long context
        {"name": "gqa_b1_l8192", "entry": "decode", "B": 1, "H_Q": 64, "H_KV": 8, "L": 8192},
        # wide groups (64 query heads per KV head), middling batch, odd length, no workspace
        {"name": "wide_b6_l3001_noalloc", "entry": "noalloc", "B": 6, "H_Q": 128, "H_KV": 2, "L": 3001},
        # a short mixed batch of chat turns, packed
        {"name": "varlen_b16_to512", "entry": "varlen", "B": 16, "H_Q": 32, "H_KV": 4,
         "lens": "uniform", "len_lo": 32, "len_hi": 512, "len_seed": 4000},
        # a loaded server's packed batch, lengths between 1 and 16 thousand
        {"name": "varlen_b32_to16k", "entry": "varlen", "B": 32, "H_Q": 64, "H_KV": 8,
         "lens": "uniform", "len_lo": 1024, "len_hi": 16384, "len_seed": 2024},
        # the same kind of load in a paged cache: most sequences short, a few long
        {"name": "paged_b64_lognormal", "entry": "paged", "B": 64, "H_Q": 32, "H_KV": 4, "page": 64,
         "lens": "lognormal", "len_lo": 16, "len_hi": 32768, "len_seed": 102},
        # the mixed batch whose host knows the lengths and keeps a schedule for it
        {"name": "scheduled_b32_to16k", "entry": "scheduled", "B": 32, "H_Q": 64, "H_KV": 8, "page": 0,
         "lens": "uniform", "len_lo": 1024, "len_hi": 16384, "len_seed": 2024},
        # many MQA sequences of mixed length, paged, scheduled
        {"name": "scheduled_mqa_b128_paged", "entry": "scheduled", "B": 128, "H_Q": 8, "H_KV": 1, "page": 128,
         "lens": "lognormal", "len_lo": 16, "len_hi": 32768, "len_seed": 106},
        # chunk states of one rank's share of long sequences, and their merge
        {"name": "partials_b8_l4093_s6", "entry": "partials", "B": 8, "H_Q": 32, "H_KV": 2, "L": 4093, "splits": 6},
        # the largest: 32 sequences of 8192 keys, 1 GiB of K/V
        {"name": "highload_b32_l8192", "entry": "decode", "B": 32, "H_Q": 64, "H_KV": 8, "L": 8192},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    while True:
        entry = rng.choice(["decode", "decode", "noalloc", "varlen", "varlen", "paged", "paged", "scheduled",
                            "scheduled", "partials", "step"])
        H_Q, H_KV = rng.choice(HEADS)
        case = {"entry": entry, "B": _log_int(rng, 1, 128), "H_Q": H_Q, "H_KV": H_KV}
        if entry in ("varlen", "paged", "scheduled"):
            hi = _log_int(rng, 256, 32768)
            case.update(lens=rng.choice(["uniform", "lognormal", "bimodal"]),
                        len_lo=rng.choice([1, 16, max(1, hi // 16)]), len_hi=hi, len_seed=rng.randrange(1 << 20))
            if entry != "varlen":
                case["page"] = rng.choice([32, 64, 128, 256] + ([0] if entry == "scheduled" else []))
        else:
            case["L"] = _log_int(rng, 33, 32768)
        if entry == "partials":
            case["splits"] = rng.randint(2, 16)
        if entry == "step":
            case["layers"] = rng.choice([16, 32, 48, 80])
            case["B"] = min(case["B"], 16)
        if _kv_bytes(case) <= MAX_KV_BYTES:
            return case


def _lengths(case):
    if "L" in case:
        return [case["L"]] * case["B"]
    rng = np.random.default_rng(case["len_seed"])
    B, lo, hi = case["B"], case["len_lo"], case["len_hi"]
    if case["lens"] == "uniform":
        x = rng.integers(lo, hi + 1, B)
    elif case["lens"] == "lognormal":
        x = np.clip(rng.lognormal(math.log(max(lo, hi / 16)), 1.0, B), lo, hi)
    else:  # bimodal: one sequence in eight at the full length, the others at a thirty-second of it
        x = np.where(rng.permutation(B) < max(1, B // 8), hi, max(lo, hi // 32))
    return [int(v) for v in x]


def _kv_bytes(case):
    return sum(_lengths(case)) * case["H_KV"] * D * 2 * 2 * case.get("layers", 1)


def _normal(g, shape, scale=1.0):
    x = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    return x.normal_(0.0, scale, generator=g)


def _tensors(case, seed):
    """The tensors of a call: q, k, v in the entry's layout, and its lengths' metadata."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    B, H_Q, H_KV = case["B"], case["H_Q"], case["H_KV"]
    lens = _lengths(case)
    t = {"lens": lens}
    if case["entry"] == "step":
        n = case["layers"]
        t["q"] = _normal(g, (n, B, H_Q, D), 2.0)
        t["k"] = _normal(g, (n, B, case["L"], H_KV, D))
        t["v"] = _normal(g, (n, B, case["L"], H_KV, D))
        return t
    t["q"] = _normal(g, (B, H_Q, D), 2.0)
    if "L" in case:
        shape = (B, case["L"], H_KV, D)
    elif case.get("page"):
        page = case["page"]
        pages = [-(-n // page) for n in lens]
        spare = 8
        shape = (sum(pages) + spare, page, H_KV, D)
        cpu = torch.Generator()
        cpu.manual_seed(seed + 1)
        order = torch.randperm(shape[0], generator=cpu, dtype=torch.int64).to(torch.int32)
        table = torch.zeros(B, max(pages), dtype=torch.int32)
        at = 0
        for b, n in enumerate(pages):
            table[b, :n] = order[at:at + n]
            at += n
        t["table"] = table.to(DEV)
        t["seq_lens"] = torch.tensor(lens, dtype=torch.int32, device=DEV)
    else:
        shape = (sum(lens), H_KV, D)
        t["cu"] = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device=DEV)
    t["k"] = _normal(g, shape)
    t["v"] = _normal(g, shape)
    return t


def prepare(case, seed):
    s = _tensors(case, seed)
    s["entry"] = case["entry"]
    s["L_max"] = max(s["lens"])
    B, H_Q, H_KV = case["B"], case["H_Q"], case["H_KV"]
    if case["entry"] == "step":
        s["out"] = torch.empty_like(s["q"])
        plan = da.da_make_plan(B, H_Q, H_KV, case["L"], policy=da.POLICY_STREAMED)
        need = da.da_workspace_bytes(B, H_Q, D, plan.num_splits)
        s["workspace"] = torch.zeros(max(need, 256), dtype=torch.uint8, device=DEV)
        s["graph"] = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(s["graph"]):
            for i in range(case["layers"]):
                da.da_decode_attn_planned(s["q"][i], s["k"][i], s["v"][i], plan, out=s["out"][i],
                                          workspace=s["workspace"])
        return s
    s["lse"] = torch.empty(B, H_Q, dtype=torch.float32, device=DEV)
    if case["entry"] == "noalloc":
        s["out"] = torch.empty(B, H_Q, D, dtype=torch.bfloat16, device=DEV)
    if case["entry"] == "scheduled":
        s["sched"], meta = da.da_make_schedule(s["lens"], H_Q, H_KV, s["L_max"])
        s["meta"] = meta.to(DEV)
    if case["entry"] == "partials":
        s["splits"] = case["splits"]
    return s


def run(s):
    entry = s["entry"]
    if entry == "step":
        s["graph"].replay()
        return s["out"]
    q, k, v, lse = s["q"], s["k"], s["v"], s["lse"]
    if entry == "decode":
        return da.da_decode_attn(q, k, v, lse_out=lse), lse
    if entry == "noalloc":
        return da.da_decode_attn_noalloc(q, k, v, out=s["out"], lse_out=lse), lse
    if entry == "varlen":
        return da.da_decode_attn(q, k, v, s["cu"], lse_out=lse, L_K_max=s["L_max"]), lse
    if entry == "paged":
        return da.da_decode_attn_paged(q, k, v, s["table"], s["seq_lens"], s["L_max"], lse_out=lse), lse
    if entry == "scheduled":
        if "table" in s:
            return da.da_decode_attn_scheduled(q, k, v, s["sched"], s["meta"], block_table=s["table"],
                                               seq_lens=s["seq_lens"], lse_out=lse), lse
        return da.da_decode_attn_scheduled(q, k, v, s["sched"], s["meta"], s["cu"], lse_out=lse), lse
    o, m, l = da.da_split_partials(q, k, v, num_splits=s["splits"], pack_gqa=1)
    return da.da_combine_splits(o, m, l, lse_out=lse), lse, o, m, l


def work(case):
    keys = sum(_lengths(case))
    layers = case.get("layers", 1)
    rows = case["B"] * case["H_Q"]
    nbytes = _kv_bytes(case) + layers * 2 * rows * D * 2
    if case["entry"] != "step":
        nbytes += rows * 4
    if case["entry"] == "partials":  # the states are written, and read again by the merge
        nbytes += 2 * case["splits"] * rows * (D + 2) * 4
    return {"bytes": nbytes, "flops": 4 * layers * keys * case["H_Q"] * D}


def tolerance(case):
    # bf16 inputs and output, probabilities in bf16 before the second product, sums in 32 bits: 1.7-1.9e-3
    # off 64 bits in every entry; four times that
    return {"rel": 8e-3}


def _attend(q, k, v):
    """q [H_Q, D], k and v [L, H_KV, D] in 64 bits: (out, lse, chunk's O~, m, l) over these keys."""
    H_Q, H_KV = q.shape[0], k.shape[1]
    qg = q.view(H_KV, H_Q // H_KV, D)
    s = torch.matmul(qg, k.permute(1, 2, 0).contiguous()) / math.sqrt(D)
    m = s.amax(dim=-1)
    p = torch.exp(s - m[..., None])
    l = p.sum(dim=-1)
    o = torch.matmul(p, v.permute(1, 0, 2).contiguous())
    return (o / l[..., None]).reshape(H_Q, D), (m + torch.log(l)).reshape(H_Q), o.reshape(H_Q, D), \
        m.reshape(H_Q), l.reshape(H_Q)


def exact(case, seed):
    t = _tensors(case, seed)
    B, H_KV = case["B"], case["H_KV"]
    q, k, v, lens = t["q"], t["k"], t["v"], t["lens"]
    if case["entry"] == "step":
        return torch.stack([torch.stack([_attend(q[i, b].double(), k[i, b].double(), v[i, b].double())[0]
                                         for b in range(B)]) for i in range(case["layers"])])

    def rows(x, b):
        if "L" in case:
            return x[b]
        if case.get("page"):
            n = -(-lens[b] // case["page"])
            return x[t["table"][b, :n].long()].reshape(-1, H_KV, D)[:lens[b]]
        at = sum(lens[:b])
        return x[at:at + lens[b]]

    got = [_attend(q[b].double(), rows(k, b).double(), rows(v, b).double()) for b in range(B)]
    out, lse = (torch.stack([r[i] for r in got]) for i in (0, 1))
    if case["entry"] != "partials":
        return out, lse
    s, L = case["splits"], case["L"]
    parts = []
    for i in range(s):
        lo, hi = i * L // s, (i + 1) * L // s
        parts.append([_attend(q[b].double(), k[b, lo:hi].double(), v[b, lo:hi].double())[2:] for b in range(B)])
    o, m, l = (torch.stack([torch.stack([r[i] for r in row]) for row in parts]) for i in range(3))
    return out, lse, o, m, l
