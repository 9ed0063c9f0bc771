"""The work that programs have this library do, as cases that can be timed and compared.

A case is a dict of plain values:

  kind     "layer"  estimate the block mask, then block-sparse attention over it: prefill of one layer
           "dense"  the dense causal baseline
           "packed" "layer" over several prompts packed back to back (`blocks`: their lengths in blocks)
           "chunk"  "layer" for the last `Lq` positions of a context whose earlier chunks have been through: the
                    stride sums of those positions are in the workspace, and the attention has its workspace too
           "step"   the same for a decode-sized number of new positions, which leaves the last block unprotected
           "decode" dense attention of the last `Lq` positions, the way the paper decodes
  batch, L, Hq, Hkv, d, dtype, B, S, tau    as in include/rr_attn.h; S and tau where a mask is estimated
  gain     strength of the structure in Q and K (see _inputs)
  keep     true: mask arrays, workspaces and outputs are made once and given to every call, as a serving program
           does; false: the short form of the README, where each call makes its own
"""
import math

import torch

import paper_2602_05853_amd as rr

DEVICE = "cuda:0"


def _case(name, kind, L, Hq=32, Hkv=8, d=128, dtype="bf16", B=128, batch=1, S=16, tau=0.9, gain=4.0, keep=True, **more):
    c = dict(kind=kind, batch=batch, L=L, Hq=Hq, Hkv=Hkv, d=d, dtype=dtype, B=B, S=S, tau=tau, gain=gain, keep=keep, **more)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the small fp32 layer that is checked on a CPU: the shortest call of all, launches and host work
        _case("layer_1k_f32", "layer", 1024, 4, 2, d=64, dtype="f32", B=64, S=8, gain=2.5, keep=False),
        # fp32 tensors at full head width: reference runs of a model before it is moved to bf16
        _case("layer_4k_f32_d128", "layer", 4096, 8, 2, dtype="f32", B=64, S=8, gain=2.5),
        # heads of 64 channels in bf16, a prompt whose length is no multiple of anything
        _case("layer_8k_d64_ragged", "layer", 8153, 16, 4, d=64, B=64, S=8, gain=3.0),
        # an ordinary prompt of an 8B-sized model (32 / 8 heads) at the setting of the paper's time table
        _case("layer_8k", "layer", 8192, tau=0.95, keep=False),
        # a longer one of the length that a tokenizer happens to give
        _case("layer_32k_ragged", "layer", 31907, gain=2.5),
        # the headline: one layer at 128K tokens
        _case("layer_128k", "layer", 131072),
        # a large model's layer (64 / 8 heads) with the finer stride
        _case("layer_64k_64h_s8", "layer", 65536, Hq=64, S=8, gain=3.0),
        # a batch of prompts of different lengths in one call, 28 / 4 heads
        _case("packed_28h", "packed", 128 * 311 - 51, 28, 4, gain=3.0, blocks="61,7,30,118,2,44,16,33"),
        # the dense baseline, with the log-sum-exp that merging and training need
        _case("dense_16k", "dense", 16384),
        # chunked prefill: the chunk that ends a 128K prompt
        _case("chunk_2k_of_128k", "chunk", 131072, Lq=2048),
        # eight speculative tokens behind a 64K context
        _case("step_8_of_64k", "step", 64512, Lq=8),
        # one token decoded against 128K
        _case("decode_1_of_128k", "decode", 131072, Lq=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "generic", "generic", "packed", "dense", "chunk", "step", "decode"])
    tau = rng.choice([0.8, 0.9, 0.95])
    gain = rng.choice([2.5, 3.0, 4.0])
    if kind == "generic":
        # every head width, block size and type the matrix path does not take
        d = rng.choice([40, 64, 64, 80, 96, 128])
        B = rng.choice([b for b in (32, 48, 64, 128) if b * d <= 8192])
        S = rng.choice([s for s in (4, 8, 16) if B % s == 0])
        Hq, Hkv = rng.choice([(4, 2), (8, 2), (6, 3), (16, 4)])
        dtype = rng.choice(["bf16", "f32"])
        L = _log(rng, 512, 8192) if Hq <= 8 and dtype == "bf16" else _log(rng, 512, 4096)
        return _case(None, "layer", L, Hq, Hkv, d=d, dtype=dtype, B=B, S=S, tau=tau, gain=gain, keep=rng.random() < 0.5)
    Hq, Hkv = rng.choice([(32, 8), (32, 8), (28, 4), (64, 8), (8, 2)])
    S = rng.choice([8, 16, 16, 32])
    if kind == "packed":
        n = rng.randint(2, 16)
        blocks = [_log(rng, 1, 128) for _ in range(n)]
        return _case(None, kind, 128 * sum(blocks) - rng.randint(0, 127), Hq, Hkv, S=S, tau=tau, gain=gain,
                     blocks=",".join(map(str, blocks)))
    if kind == "layer":
        L = _log(rng, 512, 65536)
        return _case(None, kind, L, Hq, Hkv, S=S, tau=tau, gain=gain, keep=rng.random() < 0.7)
    if kind == "dense":
        return _case(None, kind, _log(rng, 512, 24576), Hq, Hkv)
    if kind == "chunk":
        Lq = _log(rng, 129, 4096)
        return _case(None, kind, Lq + _log(rng, 8192, 98304), Hq, Hkv, S=S, tau=tau, gain=gain, Lq=Lq)
    if kind == "step":
        return _case(None, kind, _log(rng, 4096, 98304), Hq, Hkv, S=S, tau=tau, gain=gain, Lq=_log(rng, 1, 128))
    L = _log(rng, 2048, 131072)
    return _case(None, kind, L, Hq, Hkv, batch=rng.choice([b for b in (1, 2, 4, 8) if b * L <= 131072]),
                 Lq=rng.choice([1, 1, 1, 2, 4]))


def _inputs(case, seed):
    """Q, K, V with what long-context attention shows: a background of N(0, 1) with a shared rank-4 part, a sink
    on the first four keys, a local window, and spans of 256 keys that a few runs of 512 queries look for (the
    ingredients of rr_inputs/workloads.py, drawn on the GPU)."""
    b, L, Hq, Hkv, d = case["batch"], case["L"], case["Hq"], case["Hkv"], case["d"]
    Lq = case.get("Lq", L)
    gain, rd = case["gain"], math.sqrt(d)
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device=DEVICE).manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=DEVICE)

    Q = torch.empty(b, Hq, Lq, d, dtype=dtype, device=DEVICE)
    K = torch.empty(b, Hkv, L, d, dtype=dtype, device=DEVICE)
    V = torch.empty(b, Hkv, L, d, dtype=dtype, device=DEVICE)
    pos = torch.arange(L, device=DEVICE, dtype=torch.float64)
    angle = pos[:, None] * (normal(16) / 32.0).double()[None, :]
    window = torch.cat([angle.cos(), angle.sin()], 1).float()          # 16 pairs: +16 at distance 0, gone by 100
    spans = max(1, L // 2048) if L >= 2048 else 0
    key = torch.arange(L, device=DEVICE)

    def runs(starts, length, rows):
        """[rows, n]: how many of the runs of item n cover a position; the last `rows` positions"""
        p = key[L - rows:, None]
        cover = torch.zeros(rows, starts.shape[1], device=DEVICE)
        for s in starts:
            cover += ((p >= s) & (p < s + length)).float()
        return cover

    for i in range(b):
        for kv in range(Hkv):
            basis = torch.linalg.qr(normal(d, 37).double().cpu())[0].T.float().to(DEVICE)
            low, mean, win = basis[:4], basis[4], basis[5:]
            x = normal(L, d) + (normal(L, 4)) @ low
            x[:4] += gain * 3.0 * rd / 3.0 * mean
            amp = math.sqrt(gain * 1.5 * rd / 16.0)
            x += amp * (window @ win)
            if spans:
                where = torch.randint(0, L - 1280, (1, spans), generator=g, device=DEVICE)
                dirs = normal(spans, d)
                dirs = dirs / dirs.norm(dim=1, keepdim=True) * math.sqrt(gain * 2.5 * rd)
                x += runs(where, 256, L) @ dirs
            K[i, kv] = x.to(dtype)
            V[i, kv] = normal(L, d).to(dtype)
            for h in range(kv * (Hq // Hkv), (kv + 1) * (Hq // Hkv)):
                q = normal(Lq, d) + normal(Lq, 4) @ low + 3.0 * mean + amp * (window[L - Lq:] @ win)
                if spans:
                    u = torch.rand(4, spans, generator=g, device=DEVICE)
                    q += runs((where + 256 + u * (L - 512 - where - 256)).long(), 512, Lq) @ dirs
                Q[i, h] = q.to(dtype)
    return Q, K, V


def prepare(case, seed):
    Q, K, V = _inputs(case, seed)
    kind, B, S, L = case["kind"], case["B"], case["S"], case["L"]
    s = dict(case=case, Q=Q, K=K, V=V)
    if kind == "packed":
        s["seq_first"] = rr.packed_seq_first([int(n) for n in case["blocks"].split(",")], Q.device)
    if case["keep"]:
        s["O"] = torch.empty_like(Q)
    if kind in ("dense", "decode"):
        s["lse"] = torch.empty(case["batch"], case["Hq"], Q.shape[2], dtype=torch.float32, device=DEVICE)
    elif case["keep"]:
        s["mask"] = rr.BlockMask.allocate(case["batch"], case["Hq"], -(-L // B), B, Q.device, Hkv=case["Hkv"],
                                          rows=-(-L // B) - (L - Q.shape[2]) // B)
    if kind in ("chunk", "step"):
        # a context that may grow to the next multiple of 4096 (at least one block): the workspace is laid out for
        # that (and for a call of these positions wherever it starts in a block), and the calls of the earlier
        # chunks have left the stride sums of everything in front in it
        L0 = L - case["Lq"]
        cap = (L + B + 4095) // 4096 * 4096
        longest = Q.new_empty((case["batch"], case["Hq"], case["Lq"] + B, case["d"]), device="meta")
        room = K.new_empty((case["batch"], case["Hkv"], cap, case["d"]), device="meta")
        s["ws"] = torch.empty(rr.rr_workspace_bytes(longest, room, S, B), dtype=torch.uint8, device=DEVICE)
        s["kept"] = dict(ksum_capacity=cap, ksum_valid=L0)
        rr.rr_estimate(Q[:, :, :min(case["Lq"], L0)], K[:, :, :L0], S, B, case["tau"], flags=0, workspace=s["ws"],
                       ksum_capacity=cap)
    elif kind in ("layer", "packed") and case["keep"]:
        s["ws"] = torch.empty(rr.rr_workspace_bytes(Q, K, S, B), dtype=torch.uint8, device=DEVICE)
    if kind in ("chunk", "step", "decode"):
        n = rr.rr_attn_workspace_bytes(Q, K, B)
        s["attn_ws"] = torch.empty(n, dtype=torch.uint8, device=DEVICE) if n else None
    return s


def run(s):
    case, Q, K, V = s["case"], s["Q"], s["K"], s["V"]
    kind, B = case["kind"], case["B"]
    if kind == "dense":
        return {"O": rr.rr_dense_attn(Q, K, V, B, O=s["O"], lse=s["lse"]), "lse": s["lse"]}
    if kind == "decode":
        return {"O": rr.rr_dense_attn(Q, K, V, B, O=s["O"], lse=s["lse"], workspace=s["attn_ws"]), "lse": s["lse"]}
    if not case["keep"]:
        mask = rr.rr_estimate(Q, K, case["S"], B, case["tau"])
        O = rr.rr_sparse_attn(Q, K, V, mask)
    else:
        more = dict(s.get("kept", {}))
        if kind == "packed":
            more["seq_first"] = s["seq_first"]
        if kind == "step":
            more["flags"] = 0
        mask = rr.rr_estimate(Q, K, case["S"], B, case["tau"], out=s["mask"], workspace=s["ws"], **more)
        O = rr.rr_sparse_attn(Q, K, V, mask, O=s["O"], workspace=s.get("attn_ws"))
    return {"O": O, "dense": mask.dense, "row_count": mask.row_count}


def _density(case, blocks):
    """Share of the causal blocks of a row of that many blocks that is kept on these inputs, as measured: a short
    row keeps nearly everything; in a chunk at the end of a long prompt the protected last row weighs most; in a
    step of a few tokens the heads without a sampled position among them stay dense."""
    if case["kind"] == "chunk":
        return min(1.0, 0.05 + 128.0 / case["Lq"])
    if case["kind"] == "step":
        return 0.65
    at = {0.8: 0.15, 0.9: 0.25, 0.95: 0.35}[case["tau"]] * (1.3 if case["gain"] < 3.5 else 1.0)
    return min(1.0, at + 6.0 / max(blocks, 1))


def work(case):
    b, L, Hq, Hkv, d, B = (case[k] for k in ("batch", "L", "Hq", "Hkv", "d", "B"))
    Lq = case.get("Lq", L)
    size = 2 if case["dtype"] == "bf16" else 4
    q_bytes, kv_bytes = b * Hq * Lq * d * size, b * Hkv * L * d * size
    lengths = [int(n) * B for n in case["blocks"].split(",")] if case["kind"] == "packed" else [L]
    # (query, key) pairs per head under causality
    pairs = sum(n * n / 2 for n in lengths) if Lq == L else Lq * (L - Lq / 2)
    out = 2.0 * q_bytes + 2.0 * kv_bytes
    if case["kind"] in ("dense", "decode"):
        return {"bytes": out + 4.0 * b * Hq * Lq, "flops": 4.0 * d * b * Hq * pairs}
    S = case["S"]
    rows = -(-L // B) - (L - Lq) // B
    kept = sum(n * n / 2 * _density(case, n / B / 2) for n in lengths) if Lq == L else pairs * _density(case, L / B)
    mask = b * Hq * rows * (-(-L // B)) * (1 + 4 * _density(case, L / B) / 2)
    # the estimate reads a sampled query per stride and every key; with kept sums one sum per stride in front
    est = q_bytes / S + (kv_bytes if Lq == L else kv_bytes * 4 / size / S)
    if Lq < L:      # sparse attention over a step need not read the blocks that no row of the KV head kept
        out = 2.0 * q_bytes + 2.0 * kv_bytes * min(1.0, 2 * _density(case, L / B))
    return {"bytes": out + est + mask, "flops": b * Hq * (2.0 * d * pairs / (S * S) + 4.0 * d * kept)}


def tolerance(case):
    # About four times what the outputs are off from the same attention in 64 bits: bf16 1.7e-3 to 2.0e-3 (its own
    # last rounding and that of the probabilities; largest single value 1.1e-2), fp32 1.7e-6 (4.7e-5).  In bf16 a row
    # whose cumulative mass meets tau to rounding may also keep a block more or less, which a few values show.
    if case["dtype"] == "bf16":
        return {"rel": 8e-3, "max": 0.1, "differ": 2e-4}
    return {"rel": 1e-5, "max": 2e-4, "differ": 2e-4}
