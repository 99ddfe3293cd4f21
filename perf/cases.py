"""What a user of this library has it do on the GPU, as cases that can be timed and compared.

A case is one serving-loop call on a handle whose table is warm: the logits of a verification are in device
memory (the target model has just written them), contexts and the pending draft are the handle's.  Four kinds of
pass ("op"):

  step    stand_step: verify the pending tree, merge the accepted path, draft the next tree (the method's loop)
  split   the same loop through its separate entry points: stand_verify, stand_update, stand_draft
  verify  stand_verify and stand_row_results: a server that also returns the K best log-probabilities of every row
  ingest  stand_update with given rows, then stand_draft: an existing transcript goes into the table, one row per
          token of a chain of nodes
  draft   stand_draft and stand_tree_packing: a tree and its attention mask, as after a prompt or a beam copy

The workloads are those of `synth` (token streams with repeated spans; N(0, 3) noise with a few peaked tokens per
row).  `tensors` logits tensors are recorded over real steps, each peaked on the children that were pending then, and
are replayed in turn with the recorded stream tokens committed; `forces` recorded commits are used in turn, and the
recording is repeated `rounds` times with the trees that are drafted by then (deeper ones each time).  With
tensors == forces a context always sees the same row again (drafts are accepted often); with two different numbers
each context's entry is a mean over several rows (drafts are accepted seldom, as on the streams themselves).
"""
import math

import numpy as np
import torch

from paper_2506_04708_amd import binding, synth

_WARM = 48  # untimed passes of a new state: every context of the replay has been merged, the automatic plan has settled


def _case(name, op, B, V, N, D, fan, K, omax, T, dtype="bf16", log2cap=20, tensors=4, forces=5, peak=8.0, peaks=4, rho=0.5,
          shared=0, rounds=1):
    return dict(name=name, op=op, B=B, V=V, N=N, D=D, fan=fan, K=K, omax=omax, T=T, dtype=dtype, log2cap=log2cap, tensors=tensors,
                forces=forces, peak=peak, peaks=peaks, rho=rho, shared=shared, rounds=rounds)


def listed():
    return [
        # one short request on a small model, fp32 logits: nothing but launches and dependent round trips
        _case("step_tiny", "step", 1, 32000, 16, 4, "4-2-1-1", 10, 3, 0.6, "f32", 12),
        # one request on a 7B model of a 152k vocabulary: latency of a single-user server
        _case("step_single", "step", 1, 152064, 32, 6, "4-2-2-1", 10, 4, 0.6),
        # a few requests, a vocabulary whose rows start at every alignment, through the separate entry points
        _case("split_odd", "split", 6, 50257, 40, 6, "6-3-2-1", 10, 4, 0.7, "bf16", 18, 3, 3, 10.0, 2, rounds=3),
        # a small batch: 256 rows
        _case("step_batch8", "step", 8, 128256, 32, 6, "4-2-2-1", 10, 4, 0.6),
        # best-of-32 on one table, drafts seldom accepted: the benchmark's default workload
        _case("step_best32", "step", 32, 152064, 64, 8, "8-4-2-1", 16, 4, 0.6, "bf16", 22),
        # the same shape with confident targets: long accepted paths, deep drafts
        _case("step_best32_deep", "step", 32, 152064, 64, 8, "8-4-2-1", 16, 4, 0.6, "bf16", 22, 3, 3, 14.0, 1, rounds=8),
        # best-of-64 from one shared prompt, T = 1
        _case("step_best64", "step", 64, 128256, 48, 7, "6-3-2-1", 10, 4, 1.0, "bf16", 23, 4, 5, 8.0, 4, 0.6, 64),
        # tree search over 128 beams: the largest step (5 GB of logits)
        _case("step_beams128", "step", 128, 152064, 128, 10, "8-4-2-1", 32, 5, 0.8, "bf16", 22, 2, 3),
        # the heuristic initial tree of the tree optimisation
        _case("step_tree625", "step", 4, 152064, 625, 20, "initial", 16, 4, 0.6, "bf16", 20, 2, 3),
        # a server that returns log-probabilities: fp32 logits, odd vocabulary
        _case("verify_logprobs", "verify", 12, 32003, 48, 7, "6-3-2-1", 20, 4, 1.0, "f32", 18, 2, 2, 10.0, 3),
        # transcripts of four earlier trajectories go into the table, 32 tokens of each per call
        _case("ingest", "ingest", 4, 152064, 32, 31, "chain", 16, 4, 0.6, "bf16", 20, 3, 3),
        # trees for a batch, before the target model's pass
        _case("draft_packing", "draft", 32, 32768, 64, 8, "8-4-2-1", 16, 4, 0.6, "bf16", 20, 3, 3, 14.0, 1, rounds=8),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step", "step", "step", "step", "step", "split", "verify", "ingest", "draft"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    V = _log_uniform(rng, 8000, 200000)
    if rng.random() < 0.5:
        V -= V % 64
    K = rng.choice([8, 10, 16, 20, 32])
    deep = rng.random() < 0.4
    B = _log_uniform(rng, 1, 128)
    if op == "ingest":
        B = min(B, 32)
        D = rng.randint(7, 31)
        N, fan = D + 1, "chain"
    else:
        D = rng.randint(4, 10)
        fan = rng.choice(["4-2-1-1", "4-2-2-1", "6-3-2-1", "8-4-2-1"])
        f = [int(x) for x in fan.split("-")]
        most = 1 + f[0] + f[0] * f[1] * (1 + f[2] * (D - 2))
        N = _log_uniform(rng, min(most, 1 + f[0] + D), min(most, 160))
    # no more logits than the largest listed case has
    room = 128 * 128 * 152064 * 2
    while B * N * V * (2 if dtype == "bf16" else 4) > room:
        B //= 2
    rows = B * N
    log2cap = rng.choice([18, 20] if rows < 2000 else [20, 22])
    n = rng.choice([(3, 3), (2, 2)] if deep else [(4, 5), (2, 3)])
    return {k: v for k, v in _case("", op, B, V, N, D, fan, K, rng.choice([3, 4, 4, 5]), rng.choice([0.6, 0.6, 0.8, 1.0]), dtype, log2cap,
                                   n[0] if rows * V < 2 ** 30 else 2, n[1], rng.choice([12.0, 14.0]) if deep else 8.0, 1 if deep else 4,
                                   rng.choice([0.3, 0.5, 0.7]), 0, rng.choice([2, 4, 8]) if deep else 1).items() if k != "name"}


def _parent(case):
    if case["fan"] == "chain":
        return np.arange(-1, case["N"] - 1, dtype=np.int32)
    if case["fan"] == "initial":
        return binding.tree_initial(case["D"])
    return synth.make_tree(case["N"], case["D"], [int(x) for x in case["fan"].split("-")])


def _logits(case, w, step, draft_host, gen):
    """[B, N, V] on the GPU: N(0, 3) noise, +peak on each row's peaked tokens."""
    B, N, V = w.B, w.N, w.V
    peaks = torch.from_numpy(w.peaks(step, draft_host)).cuda()
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    out = torch.empty((B, N, V), device="cuda", dtype=dt)
    part = max(1, (1 << 30) // (N * V))
    for b0 in range(0, B, part):
        b1 = min(B, b0 + part)
        x = torch.randn((b1 - b0, N, V), generator=gen, device="cuda", dtype=torch.float32)
        x.mul_(3.0 ** 0.5)
        pk = peaks[b0:b1]
        x.scatter_add_(2, pk.clamp(min=0), torch.where(pk >= 0, case["peak"], 0.0).to(torch.float32))
        out[b0:b1].copy_(x)
    return out


def prepare(case, seed):
    """A handle in the middle of its run: contexts set, table warm, a draft pending; recorded logits and commits."""
    seed = int(seed)
    parent = _parent(case)
    prompt = max(16, case["shared"])
    n_rec = max(case["tensors"], case["forces"])
    w = synth.Workload(None, B=case["B"], V=case["V"], dtype=case["dtype"], N=case["N"], D=case["D"], parent=parent, K=case["K"],
                       T=case["T"], rho=case["rho"], seed=synth.BASE_SEED + seed, prompt_len=prompt, shared_prefix=case["shared"],
                       cross=0.6 if case["shared"] else 0.0, max_peaks=case["peaks"],
                       stream_len=prompt + (case["D"] + 1) * n_rec + case["D"] + 2)
    h = binding.Stand(w.V, w.B, 1, case["omax"], w.K, parent, w.T, 1 << case["log2cap"], 64, synth.BASE_SEED + seed,
                      binding.STAND_BF16 if case["dtype"] == "bf16" else binding.STAND_F32)
    gen = torch.Generator(device="cuda").manual_seed(seed & 0x7FFFFFFF)
    for b in range(w.B):
        h.set_context(b, w.prompt(b))
    out_tok, out_node, out_len, draft = h.new_outputs()
    h.draft(0, draft)
    at = []   # stream positions of the recorded steps
    st = dict(case=case, h=h, out=(out_tok, out_node, out_len), draft=draft, logits=[], force=[], i=0)
    if case["op"] == "ingest":
        st["rows"] = torch.arange(w.W, dtype=torch.int32, device="cuda").repeat(w.B, 1).contiguous()
        st["lens"] = torch.full((w.B,), w.W, dtype=torch.int32, device="cuda")
    for s in range(n_rec):
        force = np.full((w.B, w.W), 0, np.int32)
        for b in range(w.B):
            nxt = w.streams[b, w.pos[b] + 1: w.pos[b] + 1 + w.W]
            force[b, : len(nxt)] = nxt
        st["force"].append(torch.from_numpy(force).cuda())
        at.append(w.pos.copy())
        if s < case["tensors"]:
            if case["op"] == "ingest":   # the transcript's own tokens are the path of the chain
                d = np.concatenate([w.streams[np.arange(w.B), w.pos][:, None], force[:, : w.N - 1]], axis=1)
            else:
                d = draft.cpu().numpy()
            st["logits"].append(_logits(case, w, s, d, gen))
        if case["op"] == "ingest":
            w.commit(np.full(w.B, w.W))
        else:
            h.step(s, st["logits"][s % case["tensors"]], out_tok, out_node, out_len, draft, st["force"][s])
            w.commit(out_len.cpu().numpy())
    st["force"] = st["force"][: case["forces"]]
    op = case["op"]
    warm = "ingest" if op == "ingest" else "step"
    for r in range(1, case["rounds"]):
        for k in range(2 * case["forces"] + case["tensors"]):
            if k >= 2 * case["forces"]:   # the trees have settled: record this turn's logits for them
                s = st["i"] % case["tensors"]
                w.pos = at[st["i"] % case["forces"]].copy()
                st["logits"][s] = _logits(case, w, 100 * r + s, draft.cpu().numpy(), gen)
            _pass(st, warm)
    for k in range(_WARM):
        _pass(st, warm)
        if k % 8 == 7:
            torch.cuda.synchronize()
    if op == "verify":   # logits that belong to the draft that now stays pending
        st["logits"] = [_logits(case, w, 10 ** 6, draft.cpu().numpy(), gen)]
    st["i"] = 1000
    return st


def _pass(st, op):
    """One call of the serving loop."""
    h, i = st["h"], st["i"]
    out_tok, out_node, out_len = st["out"]
    draft = st["draft"]
    if op == "draft":
        h.draft(i, draft)
        mask, pos = h.tree_packing()
        return draft, mask, pos
    lg = st["logits"][i % len(st["logits"])]
    if op == "verify":
        h.verify(i, lg, out_tok, out_node, out_len)
        row_max, row_sum, top_id, top_p = h.row_results()
        return dict(tok=out_tok, node=out_node, len=out_len, max=row_max, sum=row_sum, top_id=top_id, top_p=top_p)
    st["i"] = i + 1
    force = st["force"][i % len(st["force"])]
    if op == "step":
        h.step(i, lg, out_tok, out_node, out_len, draft, force)
    elif op == "split":
        h.verify(i, lg, out_tok, out_node, out_len)
        h.update(i, lg, force, out_node, out_len)
        h.draft(i + 1, draft)
    else:  # ingest
        h.update(i, lg, force, st["rows"], st["lens"])
        h.draft(i + 1, draft)
        return draft
    return out_tok, out_node, out_len, draft


def run(state):
    return _pass(state, state["case"]["op"])


def work(case):
    """Every logit is read once; per logit a scale, an exponential and an addition; outputs are written once."""
    B, N, V, K = case["B"], case["N"], case["V"], case["K"]
    rows = B * N
    if case["op"] == "draft":
        # one table entry per drafted node, tokens, proposals, mask and positions
        return {"bytes": rows * (16 + 8 * K) * 1.0 + rows * (4 + 4 + 8 * K + N + 8), "flops": rows * K * 60.0}
    logits = rows * V * (2 if case["dtype"] == "bf16" else 4)
    return {"bytes": float(logits + rows * (8 + 12 * K)), "flops": 4.0 * rows * V}


def tolerance(case):
    """Tokens, nodes, lengths, drafts and masks are whole numbers that every correct implementation finds alike.  The
    normaliser and the probabilities of all rows are 32-bit sums (measured: 1.2e-7 off their 64-bit values)."""
    return {"rel": 1e-6, "max": 1e-5, "differ": 0.0} if case["op"] == "verify" else "exact"


def exact(case, seed):
    """Row maxima, normalisers and the K best probabilities of every row in 64 bits (log-probability passes)."""
    if case["op"] != "verify":
        return None
    st = prepare(case, seed)
    lg = st["logits"][0]
    B, N, V = lg.shape
    x = lg.reshape(B * N, V)
    T = float(np.float32(case["T"]))
    row_max, row_sum, top_p = [], [], []
    for r0 in range(0, B * N, 256):
        d = x[r0: r0 + 256].double()
        m = d.max(dim=1, keepdim=True).values
        s = torch.exp((d - m) / T).sum(dim=1)
        row_max.append(m[:, 0])
        row_sum.append(s)
        top_p.append(torch.exp((torch.topk(d, case["K"], dim=1).values - m) / T) / s[:, None])
    return dict(tok=None, node=None, len=None, max=torch.cat(row_max), sum=torch.cat(row_sum), top_id=None, top_p=torch.cat(top_p))
