"""Performance cases of the dKV-Cache hot path: the calls that a user of this library makes, over the range of sizes
of its workloads, with seeded inputs on the GPU.

Three kinds of pass:
  attn   one cache update + bidirectional attention (`attn_update`): rows of q and new K/V of each sequence against a
         position-indexed cache
  steps  the leading denoising steps of a run (`DkvRun.reset` + `denoise_step`): the steps are teacher-forced, so that
         two correct implementations compute the same thing although an arg max may fall the other way in bf16; the
         last step returns its logits. Full model width, the depth cut to a few layers (each layer repeats the same work,
         and the weights of the cut model are still several times the last-level cache)
  free   a whole free-running generation (`DkvRun.generate`), fp32

    python -c "from perf import cases; print(cases.listed())"
"""
import torch

import dkv_inputs as D
import paper_2505_15781_amd as P
from dkv_inputs import configs as C
from paper_2505_15781_amd import binding

_MODELS = {"tiny": C.TINY, "llada_8b": C.LLADA_8B, "dream_7b": C.DREAM_7B}
_VARIANTS = {"decode": C.DECODE, "greedy": C.GREEDY, "prefill": C.PREFILL, "pd": C.PD}


def _attn(name, batch, q_heads, kv_heads, seq_len, rows, ragged=False, head_dim=128):
    return {"name": name, "kind": "attn", "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads, "seq_len": seq_len,
            "head_dim": head_dim, "rows": rows, "ragged": ragged}


def _steps(name, model, layers, variant, batch, prompt, gen, block, per_step, refresh, steps, window=0, shift=False):
    return {"name": name, "kind": "steps", "model": model, "layers": layers, "variant": variant, "batch": batch,
            "prompt": prompt, "gen": gen, "block": block, "per_step": per_step, "refresh": refresh, "steps": steps,
            "window": window, "shift": shift}


def listed():
    return [
        # one layer of a batch-1 generation near its end: two active rows, the smallest call there is
        _attn("attn_2rows_b1", 1, 32, 32, 512, 2),
        # the isolated cache-update + attention benchmark at a small, a middle and its largest active set
        _attn("attn_8rows", 8, 32, 32, 1024, 8),
        _attn("attn_128rows", 8, 32, 32, 1024, 128),
        _attn("attn_512rows", 8, 32, 32, 1024, 512),
        # grouped-query heads, a batch whose sequences are at different points of their schedule
        _attn("attn_gqa_ragged", 16, 28, 4, 768, 129, ragged=True),
        # a toy model in fp32, a whole generation: nothing but latency and launches
        {"name": "tiny_fp32_generation", "kind": "free", "prompt": 32, "gen": 32, "block": 32, "refresh": 8},
        # the headline workload from its start: one refresh interval, 512 rows and then 256, 255, ... rows
        _steps("decode_first_steps", "llada_8b", 8, "decode", 1, 256, 256, 32, 1, 8, 8),
        # a short answer: two refreshes, otherwise 32 rows and fewer, every step streams the weights
        _steps("decode_short_answer", "llada_8b", 8, "decode", 1, 256, 32, 32, 1, 8, 16),
        # a small batch, two tokens a step: 1536 rows once, then about 500
        _steps("decode_batch8", "llada_8b", 8, "decode", 8, 128, 64, 32, 2, 8, 8),
        # long sequences, Greedy caching: 6144 rows at the refresh, then a few rows around each commit
        _steps("greedy_long", "llada_8b", 4, "greedy", 4, 1024, 512, 64, 1, 4, 4, window=4),
        # shifted logits, the prompt cached once, sizes that divide nothing
        _steps("prefill_shift_odd", "dream_7b", 4, "prefill", 3, 197, 93, 31, 1, 8, 3, shift=True),
        # the largest: batch 16 of the 7B shape, 12288 rows at the first step, then 4096 rows and as many candidates
        _steps("pd_batch16", "dream_7b", 4, "pd", 16, 512, 256, 256, 1, 4, 4),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(lo * (hi / lo) ** rng.random() + 0.5))


def draw(rng):
    """One more case of the ranges above (no name)."""
    largest = work(listed()[-1])["flops"]
    while True:
        kind = rng.choice(("attn", "attn", "attn", "steps", "steps", "steps", "free"))
        if kind == "attn":
            q_heads, kv_heads = rng.choice(((32, 32), (32, 32), (28, 4), (16, 16), (24, 8)))
            seq_len = _log_int(rng, 64, 2048)
            c = _attn("", _log_int(rng, 1, 16), q_heads, kv_heads, seq_len, _log_int(rng, 1, max(2, seq_len // 2)),
                      rng.random() < 0.4, rng.choice((128, 128, 128, 64)))
        elif kind == "free":
            block = rng.choice((8, 16, 32))
            c = {"name": "", "kind": "free", "prompt": _log_int(rng, 4, 64), "gen": block * rng.randint(1, 64 // block),
                 "block": block, "refresh": rng.choice((2, 4, 8))}
        else:
            variant = rng.choice(("decode", "decode", "greedy", "prefill", "pd"))
            block, per_step = rng.randint(8, 64), 1
            if block % 2 == 0:
                per_step = rng.choice((1, 2))
            refresh = rng.choice((2, 4, 8))
            gen = block * rng.randint(1, 8)
            c = _steps("", rng.choice(("llada_8b", "dream_7b")), rng.randint(2, 8), variant, _log_int(rng, 1, 16),
                       _log_int(rng, 32, 1024), gen, block, per_step, refresh, min(gen // per_step, rng.randint(2, 9)),
                       rng.choice((2, 4, 6)) if variant == "greedy" else 0, rng.random() < 0.25)
            if c["batch"] * (c["prompt"] + gen) > 12288 or work(c)["flops"] > 0.5 * largest:
                continue
        del c["name"]
        return c


def _model_run(case):
    if case["kind"] == "free":
        return C.TINY, C.RunShape(batch=1, prompt_len=case["prompt"], gen_len=case["gen"], steps=case["gen"],
                                  block_len=case["block"], refresh_interval=case["refresh"], variant=C.DECODE)
    variant = _VARIANTS[case["variant"]]
    model = _MODELS[case["model"]].with_layers(case["layers"])
    run = C.RunShape(batch=case["batch"], prompt_len=case["prompt"], gen_len=case["gen"],
                     steps=case["gen"] // case["per_step"], block_len=case["block"], refresh_interval=case["refresh"],
                     variant=variant, window=case["window"], shift_logits=int(case["shift"]),
                     remask=C.RANDOM_ORDER if variant == C.GREEDY else C.CONFIDENCE)
    return model, run


def _rows_and_candidates(run, t):
    """Rows recomputed and candidates projected onto the vocabulary at step t, all sequences (an upper bound for Greedy
    windows that clip or overlap and for shifted logits)."""
    k, L, G = run.k_per_step, run.seq_len, run.gen_len
    refresh = t % run.refresh_interval == 0
    everything = t == 0 or (refresh and run.variant in (C.DECODE, C.GREEDY))
    if everything:
        rows = L
    elif run.variant == C.PREFILL or refresh:
        rows = G
    elif run.variant == C.GREEDY:
        rows = min(L, k * (run.window + 3))
    else:
        rows = G - t * k + k
    cands = min(rows, run.block_len - (t % run.steps_per_block) * k)
    if run.shift_logits and not everything:
        rows = min(L, rows + cands)
    return run.batch * rows, run.batch * cands


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "attn":
        B, Hq, Hkv, L, dh, A = (case[k] for k in ("batch", "q_heads", "kv_heads", "seq_len", "head_dim", "rows"))
        counts = torch.full((B,), A, dtype=torch.int64, device="cuda")
        if case["ragged"]:        # from A rows down to a few, the sequences in random order
            counts = (A * torch.arange(B, 0, -1, device="cuda") // B)[torch.rand(B, generator=g, device="cuda").argsort()]
        order = torch.rand((B, L), generator=g, device="cuda").argsort(dim=1)      # distinct random positions
        taken = torch.zeros((B, L), dtype=torch.bool, device="cuda")
        taken.scatter_(1, order, torch.arange(L, device="cuda")[None, :] < counts[:, None])
        idx = taken.nonzero()[:, 1].to(torch.int32).contiguous()
        off = torch.zeros(B + 1, dtype=torch.int32, device="cuda")
        off[1:] = counts.cumsum(0)
        R = int(off[-1])

        def normal(*shape):
            return torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)

        nb = P.attn_update_workspace_bytes(B, Hq, Hkv, L, dh, P.BF16, A)
        q = normal(R, Hq, dh)
        return {"k_cache": normal(B, Hkv, L, dh), "v_cache": normal(B, Hkv, L, dh), "q": q, "k_new": normal(R, Hkv, dh),
                "v_new": normal(R, Hkv, dh), "idx": idx, "off": off, "out": torch.zeros_like(q), "rows": R, "max_rows": A,
                "ws": torch.empty(max(nb, 256), dtype=torch.uint8, device="cuda")}
    model, run = _model_run(case)
    prompt = D.prompt_tokens(model, run, seed)
    if case["kind"] == "free":
        return {"run": P.DkvRun(model, run, binding.random_weights(model, seed), prompt)}
    order = D.random_block_order(run, seed)               # commits: the blocks left to right, shuffled inside
    run_handle = P.DkvRun(model, run, binding.random_weights(model, seed), prompt,
                          order=order if run.remask == C.RANDOM_ORDER else None)
    k, n = run.k_per_step, case["steps"]
    pos = torch.from_numpy(order[:, :n * k]).cuda().view(run.batch, n, k).transpose(0, 1).contiguous()
    tok = torch.randint(0, model.mask_id, (n, run.batch, k), generator=g, device="cuda", dtype=torch.int32)
    logits = torch.zeros((_rows_and_candidates(run, n - 1)[1], model.vocab), dtype=torch.float32, device="cuda")
    return {"run": run_handle, "pos": pos, "tok": tok, "steps": n, "logits": logits}


def run(state):
    if "q" in state:
        P.attn_update(state["k_cache"], state["v_cache"], state["q"], state["k_new"], state["v_new"], state["idx"],
                      state["off"], state["out"], state["rows"], state["max_rows"], P.BF16, state["ws"])
        return {"out": state["out"], "k_cache": state["k_cache"], "v_cache": state["v_cache"]}
    g = state["run"]
    g.reset()
    got = {"tokens": g.tokens, "pos": g.decoded_pos, "tok": g.decoded_tok, "conf": g.decoded_conf, "stamp": g.stamp,
           "k_cache": g.k_cache, "v_cache": g.v_cache}
    if "logits" not in state:
        g.generate()
        return got
    last = state["steps"] - 1
    for t in range(last + 1):
        g.denoise_step(t, state["pos"][t], state["tok"][t], state["logits"] if t == last else None)
    got["logits"] = state["logits"]
    return got


def work(case):
    """Attention: K/V, queries and new rows read once, outputs and replaced rows written once. Models: every step reads
    all weights (more than any cache holds between steps; the toy model's too), the embedding rows and the K/V of all
    positions, and writes the K/V of its rows; the last step writes its logits."""
    if case["kind"] == "attn":
        B, Hq, Hkv, L, dh, A = (case[k] for k in ("batch", "q_heads", "kv_heads", "seq_len", "head_dim", "rows"))
        R = sum(A * b // B for b in range(1, B + 1)) if case["ragged"] else A * B
        return {"bytes": 2.0 * dh * (2 * B * Hkv * L + 2 * R * Hq + 4 * R * Hkv), "flops": 4.0 * R * Hq * L * dh}
    m, r = _model_run(case)
    n = case.get("steps", r.steps)
    es = 4 if m.dtype == C.FP32 else 2
    qn = m.n_q_heads * m.head_dim
    layer = m.qkv_rows * m.d_model + m.d_model * qn + 3 * m.d_ffn * m.d_model
    kv = 2 * m.n_kv_heads * m.head_dim
    nbytes = flops = 0.0
    for t in range(n):
        rows, cands = _rows_and_candidates(r, t)
        nbytes += es * (m.n_layers * (layer + kv * (r.batch * r.seq_len + rows)) + m.vocab * m.d_model + rows * m.d_model)
        flops += 2.0 * rows * m.n_layers * layer + 4.0 * rows * m.n_layers * qn * r.seq_len + 2.0 * cands * m.vocab * m.d_model
    if case["kind"] == "steps":
        nbytes += 4.0 * cands * m.vocab
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Measured between two builds that add up in another order (K loops started elsewhere, keys dealt to the wavefronts
    # another way): attention 2.6e-3 and at most 1.2e-2 of a value (bf16 probabilities and output); 4 to 8 layers of
    # bf16 activations and cache 6e-3 to 1.4e-2 and at most 5.1e-2; four times that, as far as 3e-2. The fp32 model: sums
    # of up to 512 fp32 terms and an exponential.
    if case["kind"] == "attn":
        return {"rel": 1e-2, "max": 5e-2}
    if case["kind"] == "free":
        return {"rel": 1e-5, "max": 4e-4}
    return {"rel": 3e-2, "max": 0.2}
