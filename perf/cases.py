"""The performance cases of this library: what one rank's program has it do, through the public
entry points (ring.py and binding.py), from calls of a few hundred tokens to the 256K-token shards.

Kinds of case
  ring     one virtual rank's ring steps (rank_forward, and rank_backward where `backward`), on one
           or two launch lanes; `packed` runs the packed-document plan of the same ring
  shard    head-shard (Ulysses) mode: the whole packed sequence in one step, some of the heads
  block    one step call on a short query block at the end of a long key block
  combine  two partial results that arrive from elsewhere merged into a running one, the cast of the
           final O and the delta pre-pass
  move     the row permutations around the attention: `zigzag` sharding there and back, or `heads`
           packed for the all-to-all there and back
"""
import math

import numpy as np
import torch

from paper_2408_10188_amd import accounting, ring, synth
from paper_2408_10188_amd import binding as B

DEV = "cuda:0"


def listed():
    return [
        # The full-precision configuration that the parity work runs on: a few launches of little work.
        dict(name="ring_f32_tiny", kind="ring", dtype="f32", hq=2, hkv=1, d=64, n=2, c=128, rank=0, packed=False, backward=True, lanes=1),
        # A short packed sample or a debugging run: every launch is smaller than the chip, tiles are ragged.
        dict(name="ring_small_ragged", kind="ring", dtype="bf16", hq=4, hkv=2, d=128, n=2, c=160, rank=1, packed=False, backward=True, lanes=1),
        # A 16K-token prefill over four ranks: forward only, launches of about 0.1 ms.
        dict(name="ring_prefill_16k", kind="ring", dtype="bf16", hq=28, hkv=4, d=128, n=4, c=2048, rank=2, packed=False, backward=False, lanes=2),
        # Training on 64K tokens over eight ranks; the last rank's steps are short query blocks on all keys.
        dict(name="ring_train_64k", kind="ring", dtype="bf16", hq=28, hkv=4, d=128, n=8, c=4096, rank=7, packed=False, backward=True, lanes=2),
        # Training on 256K tokens over 32 ranks: the workload that bench.py reports.
        dict(name="ring_train_256k", kind="ring", dtype="bf16", hq=28, hkv=4, d=128, n=32, c=4096, rank=0, packed=False, backward=True, lanes=2),
        # The same 256K tokens on a mesh of 4 head ranks x 8 ring ranks: few heads, long chunks.
        dict(name="mesh_train_256k", kind="ring", dtype="bf16", hq=7, hkv=1, d=128, n=8, c=16384, rank=3, packed=False, backward=True, lanes=2),
        # 64K tokens packed from several long-video samples, ring steps cut at the documents.
        dict(name="ring_packed_64k", kind="ring", dtype="bf16", hq=28, hkv=4, d=128, n=8, c=4096, rank=5, packed=True, pack_seed=3, frames=128,
             backward=True, lanes=1),
        # Head-shard mode on the whole 256K-token pack: the largest call there is.
        dict(name="shard_train_256k", kind="shard", hq=7, hkv=1, tokens=262144, pack_seed=0, frames=512, backward=True, lanes=2),
        # Head-shard mode on a pack of short clips whose lengths fit no tile.
        dict(name="shard_train_20k_odd", kind="shard", hq=7, hkv=1, tokens=20011, pack_seed=5, frames=24, backward=True, lanes=1),
        # A question of some two hundred text tokens behind a 32K-token video: one forward step, few query rows.
        dict(name="block_question_32k", kind="block", hq=28, hkv=4, n_q=203, n_k=32768, backward=False),
        # Partial results of two ring neighbours combined on one rank of the 256K-token workload, then what precedes the backward.
        dict(name="combine_8k_rows", kind="combine", dtype="bf16", hq=28, d=128, rows=8192),
        # Sharding Q of the 256K-token sequence over 32 ranks and bringing it back.
        dict(name="move_zigzag_256k", kind="move", what="zigzag", tokens=262144, parts=32, heads=28, d=128),
    ]


_MOST_FLOPS = 9e13                      # the largest listed case has 9.3e13


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ring", "ring", "ring", "ring", "packed", "f32", "shard", "shard", "block", "block", "combine", "move"])
    while True:
        if kind == "f32":
            hkv = rng.choice([1, 2])
            n = rng.randint(1, 4)
            case = dict(kind="ring", dtype="f32", hq=hkv * rng.choice([1, 2, 4]), hkv=hkv, d=rng.choice([64, 128]), n=n,
                        c=_log_int(rng, 24, 400), rank=rng.randrange(n), packed=False, backward=True, lanes=1)
        elif kind in ("ring", "packed"):
            hq, hkv = rng.choice([(28, 4), (28, 4), (14, 2), (7, 1), (4, 2), (8, 8)])
            n = rng.choice([1, 2, 3, 4, 6, 8, 16])
            case = dict(kind="ring", dtype="bf16", hq=hq, hkv=hkv, d=128, n=n, c=_log_int(rng, 48, 12000), rank=rng.randrange(n),
                        packed=kind == "packed", backward=rng.random() < 0.7, lanes=1 if kind == "packed" else rng.choice([1, 2]))
            if kind == "packed":
                case.update(pack_seed=rng.randrange(1 << 20), frames=rng.choice([24, 128, 512]))
        elif kind == "shard":
            hq, hkv = rng.choice([(7, 1), (7, 1), (14, 2), (4, 2)])
            case = dict(kind="shard", hq=hq, hkv=hkv, tokens=_log_int(rng, 900, 262144), pack_seed=rng.randrange(1 << 20),
                        frames=rng.choice([24, 128, 512]), backward=rng.random() < 0.7, lanes=rng.choice([1, 2]))
        elif kind == "block":
            hq, hkv = rng.choice([(28, 4), (28, 4), (7, 1), (8, 8)])
            n_q = _log_int(rng, 1, 3000)
            case = dict(kind="block", hq=hq, hkv=hkv, n_q=n_q, n_k=n_q + _log_int(rng, 300, 120000), backward=rng.random() < 0.4)
        elif kind == "combine":
            case = dict(kind="combine", dtype=rng.choice(["bf16", "bf16", "f32"]), hq=rng.choice([28, 14, 7, 4]), d=128,
                        rows=_log_int(rng, 150, 40000))
        else:
            parts, what = rng.choice([2, 3, 4, 8, 16, 32]), rng.choice(["zigzag", "heads"])
            tokens = _log_int(rng, 800, 262144)
            case = dict(kind="move", what=what, tokens=tokens // (2 * parts) * 2 * parts if what == "zigzag" else tokens, parts=parts,
                        heads=rng.choice([28, 7, 4, 1]) if what == "zigzag" else parts * rng.choice([1, 3, 7] if parts < 8 else [1]), d=128)
        if work(case)["flops"] <= _MOST_FLOPS:
            return case


# ---- work ---------------------------------------------------------------------------------------

def _cu(case, tokens):
    return synth.packed_cu_seqlens(tokens, case["pack_seed"], frames=(4, case["frames"]))


def _row_pairs(case, tokens, pos):
    """Visible pairs per head of the query rows at positions `pos` of a packed sequence."""
    cu = _cu(case, tokens).astype(np.int64)
    return int((pos - cu[np.searchsorted(cu, pos, side="right") - 1] + 1).sum())


def _elt(case):
    return 4 if case.get("dtype", "bf16") == "f32" else 2


def _attention_work(case, q_rows, k_rows, pairs):
    """Q, K, V (dO) read once, O, LSE (dQ, dK, dV) written once."""
    hq, d, e = case["hq"], case.get("d", 128), _elt(case)
    q_side, kv_side = q_rows * hq * d, k_rows * case["hkv"] * d
    nbytes = q_side * 2 * e + kv_side * 2 * e + q_rows * hq * 4
    if case["backward"]:
        nbytes += q_side * (e + 4) + kv_side * 2 * 4
    return {"bytes": nbytes, "flops": accounting.attention_flops(pairs, d, hq, True, case["backward"])}


def work(case):
    kind = case["kind"]
    if kind == "ring":
        n, c, rank = case["n"], case["c"], case["rank"]
        pairs = accounting.zigzag_pairs_of_rank(n, c)
        if case["packed"]:
            pos = np.concatenate([np.arange(ch * c, (ch + 1) * c, dtype=np.int64) for ch in (rank, 2 * n - 1 - rank)])
            pairs = _row_pairs(case, 2 * n * c, pos)
        return _attention_work(case, 2 * c, (2 * n - rank) * c, pairs)      # no key beyond the second chunk is visible
    if kind == "shard":
        return _attention_work(case, case["tokens"], case["tokens"], accounting.packed_pairs(np.diff(_cu(case, case["tokens"]))))
    if kind == "block":
        n_q, n_k = case["n_q"], case["n_k"]
        return _attention_work(case, n_q, n_k, n_q * (n_k - n_q) + accounting.causal_pairs(n_q))
    if kind == "combine":
        e, elems, heads = _elt(case), case["rows"] * case["hq"] * case["d"], case["rows"] * case["hq"]
        # two partials and dO read; running O, final O, LSE and delta written
        return {"bytes": elems * (2 * 4 + e + 4 + e) + heads * (2 * 4 + 4 + 4), "flops": elems * 8}
    size = case["tokens"] * case["heads"] * case["d"] * 2
    return {"bytes": 4 * size, "flops": 0}


# ---- inputs -------------------------------------------------------------------------------------

def _maker(seed, dtype):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)

    def normal(*size, sigma=1.0, kind=dtype):
        x = torch.empty(size, dtype=torch.float32, device=DEV)
        return x.normal_(0.0, sigma, generator=gen).to(kind)
    return normal


def _buffers(case, s, q, kv_size, k):
    """What a rank keeps for a pass beside its inputs."""
    dev, f32 = q.device, torch.float32
    s["o_acc"] = torch.empty(q.shape, dtype=f32, device=dev)
    s["lse"] = torch.empty(q.shape[1], q.shape[0], dtype=f32, device=dev)
    s["o_final"] = torch.empty_like(q)
    if case["backward"]:
        s["delta"] = torch.empty_like(s["lse"])
        s["dq"] = torch.empty_like(s["o_acc"])
        s["dk"] = torch.zeros(kv_size, dtype=f32, device=dev)     # rows that no query of this rank sees stay zero
        s["dv"] = torch.zeros(kv_size, dtype=f32, device=dev)
    rows_k = k.shape[-3]
    s["shape"] = ring.shape_for(q, k, B.MMSP_F32 if case.get("dtype") == "f32" else B.MMSP_BF16, q.shape[0])
    s["ws_bytes"] = ring.workspace_bytes(s["shape"], q.shape[0], rows_k)
    s["ws"] = torch.empty(max(s["ws_bytes"], 16), dtype=torch.uint8, device=dev)
    s["side"] = None
    if case.get("lanes") == 2:
        s["side"] = ring.SideLane(torch.cuda.Stream(), torch.empty_like(s["o_acc"]), torch.empty_like(s["lse"]),
                                  torch.empty_like(s["ws"]), s["ws_bytes"])


def prepare(case, seed):
    kind, s = case["kind"], {"case": case}
    dtype = torch.float32 if case.get("dtype") == "f32" else torch.bfloat16
    normal = _maker(seed, dtype)
    if kind == "move":
        s["x"] = normal(case["tokens"], case["heads"], case["d"])
        s["moved"], s["back"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
        return s
    if kind == "combine":
        size = (case["rows"], case["hq"], case["d"])
        s["parts"] = [(normal(*size, kind=torch.float32, sigma=0.05), normal(size[1], size[0], kind=torch.float32, sigma=0.5) + 8.0)
                      for _ in range(2)]
        s["do"] = normal(*size)
        s["o_acc"] = torch.empty(size, dtype=torch.float32, device=DEV)
        s["lse"] = torch.empty(size[1], size[0], dtype=torch.float32, device=DEV)
        s["o_final"], s["delta"] = torch.empty_like(s["do"]), torch.empty_like(s["lse"])
        s["shape"] = ring.shape_for(s["do"], s["do"], B.MMSP_F32 if case["dtype"] == "f32" else B.MMSP_BF16, size[0])
        return s
    hq, hkv, d = case["hq"], case["hkv"], case.get("d", 128)
    sigma = 0.5 if dtype == torch.bfloat16 else 1.0
    if kind == "ring":
        q_rows, kv_size = 2 * case["c"], (case["n"], 2 * case["c"], hkv, d)
    elif kind == "shard":
        q_rows, kv_size = case["tokens"], (case["tokens"], hkv, d)
    else:
        q_rows, kv_size = case["n_q"], (case["n_k"], hkv, d)
    s["q"], s["k"], s["v"] = normal(q_rows, hq, d, sigma=sigma), normal(*kv_size, sigma=sigma), normal(*kv_size, sigma=sigma)
    if case["backward"]:
        s["do"] = normal(q_rows, hq, d)
    _buffers(case, s, s["q"], kv_size, s["k"])
    if kind == "shard" or case.get("packed"):
        s["cu_host"] = _cu(case, case["tokens"] if kind == "shard" else 2 * case["n"] * case["c"])
        s["cu"] = torch.from_numpy(s["cu_host"]).to(DEV)
        s["docs"] = len(s["cu_host"]) - 1
    if kind == "block":
        s["block"] = B.make_block(0, q_rows, 0, case["n_k"], B.MMSP_MASK_CAUSAL_DIAG, case["n_k"] - q_rows, 0)
    return s


# ---- one pass -----------------------------------------------------------------------------------

def _outputs(case, s):
    return (s["o_final"], s["lse"], s["dq"], s["dk"], s["dv"]) if case["backward"] else (s["o_final"], s["lse"])


def _run_ring(case, s, stream):
    n, rank = case["n"], case["rank"]
    T = 2 * n * case["c"]
    room = dict(ws=s["ws"], ws_bytes=s["ws_bytes"], stream=stream)
    if case["packed"]:
        ring.rank_forward_packed(s["shape"], T, n, rank, s["q"], s["k"], s["v"], s["cu"], s["docs"], s["o_acc"], s["lse"], s["o_final"],
                                 cu_host=s["cu_host"], **room)
    else:
        ring.rank_forward(s["shape"], T, n, rank, s["q"], s["k"], s["v"], s["o_acc"], s["lse"], s["o_final"], side=s["side"], **room)
    if case["backward"]:
        s["dq"].zero_()
        if case["packed"]:
            ring.rank_backward_packed(s["shape"], T, n, rank, s["q"], s["k"], s["v"], s["cu"], s["docs"], s["o_final"], s["do"], s["lse"],
                                      s["delta"], s["dq"], s["dk"], s["dv"], cu_host=s["cu_host"], **room)
        else:
            ring.rank_backward(s["shape"], T, n, rank, s["q"], s["k"], s["v"], s["o_final"], s["do"], s["lse"], s["delta"], s["dq"],
                               s["dk"], s["dv"], side=s["side"], **room)
    return _outputs(case, s)


def _run_shard(case, s, stream):
    T = case["tokens"]
    room = dict(ws=s["ws"], ws_bytes=s["ws_bytes"], stream=stream)
    ring.ulysses_forward(s["shape"], T, s["q"], s["k"], s["v"], s["cu"], s["docs"], s["o_acc"], s["lse"], s["o_final"], **room)
    if case["backward"]:
        s["dq"].zero_()
        ring.ulysses_backward(s["shape"], T, s["q"], s["k"], s["v"], s["cu"], s["docs"], s["o_final"], s["do"], s["lse"], s["delta"],
                              s["dq"], s["dk"], s["dv"], side=s["side"], **room)
    return _outputs(case, s)


def _run_block(case, s, stream):
    B.mmsp_attn_step_fwd(s["shape"], s["block"], s["q"], s["k"], s["v"], s["o_acc"], s["lse"], False, s["ws"], s["ws_bytes"], stream)
    B.mmsp_attn_merge(s["shape"], 0, case["n_q"], s["o_acc"], s["lse"], None, None, s["o_final"], stream=stream)
    if case["backward"]:
        s["dq"].zero_()
        B.mmsp_attn_step_bwd(s["shape"], s["block"], s["q"], s["k"], s["v"], s["o_final"], s["do"], s["lse"], s["delta"], True, s["dq"],
                             s["dk"], s["dv"], False, s["ws"], s["ws_bytes"], stream)
    return _outputs(case, s)


def _run_combine(case, s, stream):
    rows, do = case["rows"], s["do"]
    nothing = B.make_block(0, rows, 0, 0, B.MMSP_MASK_NONE)
    B.mmsp_attn_step_fwd(s["shape"], nothing, do, do, do, s["o_acc"], s["lse"], False, stream=stream)     # an empty running result
    for i, (o_part, lse_part) in enumerate(s["parts"]):
        B.mmsp_attn_merge(s["shape"], 0, rows, s["o_acc"], s["lse"], o_part, lse_part, s["o_final"] if i else None, stream=stream)
    B.mmsp_attn_delta(s["shape"], 0, rows, s["o_final"], do, s["delta"], stream=stream)
    return s["o_acc"], s["lse"], s["o_final"], s["delta"]


def _run_move(case, s, stream):
    T, parts, token_bytes = case["tokens"], case["parts"], case["heads"] * case["d"] * 2
    if case["what"] == "zigzag":
        B.mmsp_zigzag_gather(T, parts, token_bytes, s["x"], s["moved"], stream)
        B.mmsp_zigzag_scatter(T, parts, token_bytes, s["moved"], s["back"], stream)
    else:
        B.mmsp_a2a_pack_heads(T, parts, token_bytes // parts, s["x"], s["moved"], stream)
        B.mmsp_a2a_unpack_heads(T, parts, token_bytes // parts, s["moved"], s["back"], stream)
    return s["moved"], s["back"]


def run(state):
    case = state["case"]
    one = {"ring": _run_ring, "shard": _run_shard, "block": _run_block, "combine": _run_combine, "move": _run_move}[case["kind"]]
    return one(case, state, torch.cuda.current_stream().cuda_stream)


def tolerance(case):
    # Measured: bf16 against the float32 kernels on the same inputs and against the float64 oracle, rings of 640 to 16384 tokens
    # and a pack of short clips: rel 2.4e-3 (P, dS and the final O are rounded to bf16), max 0.14 (the first rows of a sequence
    # are far larger than the root mean square, so their rounding is too, the more the longer the sequence).  float32 against
    # the oracle: rel 8e-7, max 8e-6.
    if case["kind"] == "move":
        return "exact"
    if case["kind"] == "combine":       # float32 sums; the final O is rounded to bf16, where the last bit may go either way
        return {"rel": 2e-5, "max": 1e-4} if case["dtype"] == "f32" else {"rel": 2e-3, "max": 0.02}
    return {"rel": 1e-5, "max": 1e-4} if case.get("dtype") == "f32" else {"rel": 1e-2, "max": 0.6}


# ---- the same in 64 bits ------------------------------------------------------------------------

def _exact_attention(case, s):
    """Masked softmax attention and its gradients by their definition, one head and a few hundred query rows at a time."""
    hq, hkv, d, f64 = case["hq"], case["hkv"], case.get("d", 128), torch.float64
    q_rows = s["q"].shape[0]
    if case["kind"] == "ring":
        n, c, rank = case["n"], case["c"], case["rank"]
        chunk = torch.arange(c, device=DEV)
        k_pos = torch.cat([chunk + ch * c for r in range(n) for ch in (r, 2 * n - 1 - r)])
        q_pos = torch.cat([chunk + ch * c for ch in (rank, 2 * n - 1 - rank)])
    else:
        n_k = s["k"].shape[0]
        k_pos, q_pos = torch.arange(n_k, device=DEV), torch.arange(n_k - q_rows, n_k, device=DEV)
    order = torch.argsort(k_pos)                            # key rows in sequence order: position p is row order[p]
    first = torch.zeros_like(q_pos)
    if "cu" in s:
        cu = s["cu"].long()
        first = cu[torch.searchsorted(cu, q_pos, right=True) - 1]
    scale = 1.0 / math.sqrt(d)
    o = torch.empty(q_rows, hq, d, dtype=f64, device=DEV)
    lse = torch.empty(hq, q_rows, dtype=f64, device=DEV)
    if case["backward"]:
        dq, dk, dv = torch.empty_like(o), torch.zeros(len(order), hkv, d, dtype=f64, device=DEV), torch.zeros(len(order), hkv, d, dtype=f64, device=DEV)
    pos = torch.arange(len(order), device=DEV)
    for kv in range(hkv):
        k = s["k"].reshape(-1, hkv, d)[order, kv].to(f64)
        v = s["v"].reshape(-1, hkv, d)[order, kv].to(f64)
        for r0 in range(0, q_rows, 512):
            rows = slice(r0, min(r0 + 512, q_rows))
            lo, hi = int(first[rows].min()), int(q_pos[rows].max()) + 1
            hidden = (pos[lo:hi] > q_pos[rows, None]) | (pos[lo:hi] < first[rows, None])
            for h in range(kv * (hq // hkv), (kv + 1) * (hq // hkv)):
                q = s["q"][rows, h].to(f64)
                p = (q @ k[lo:hi].T).mul_(scale).masked_fill_(hidden, -math.inf)
                lse[h, rows] = torch.logsumexp(p, 1)
                p.sub_(lse[h, rows, None]).exp_()
                o[rows, h] = p @ v[lo:hi]
                if case["backward"]:
                    do = s["do"][rows, h].to(f64)
                    dv[lo:hi, kv] += p.T @ do
                    ds = (do @ v[lo:hi].T).sub_((do * o[rows, h]).sum(1, keepdim=True)).mul_(p).mul_(scale)
                    dq[rows, h] = ds @ k[lo:hi]
                    dk[lo:hi, kv] += ds.T @ q
    if not case["backward"]:
        return o, lse
    back = torch.argsort(order)
    return o, lse, dq, dk[back].reshape(s["k"].shape), dv[back].reshape(s["k"].shape)


def exact(case, seed):
    if case["kind"] == "move":
        return None
    s = prepare(case, seed)
    if case["kind"] != "combine":
        return _exact_attention(case, s)
    (o1, l1), (o2, l2) = [(o.double(), lse.double()) for o, lse in s["parts"]]
    lse = torch.logaddexp(l1, l2)
    o = torch.exp(l1 - lse).T[:, :, None] * o1 + torch.exp(l2 - lse).T[:, :, None] * o2
    return o, lse, o, (o * s["do"].double()).sum(2).T.contiguous()
