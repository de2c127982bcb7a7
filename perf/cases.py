"""What this library is timed on: calls as a decode loop makes them, through the package's entry points.

One decode round of adaptive speculative decoding makes up to k_max drafting calls (`draft_step`, or
`draft_entropy` where the caller has a sampler of its own) and one `verify` call that applies the round to
the adaptive state.  The cases run from one sequence (how the paper decodes) to a serving batch, over both
logit types, with padded and with odd vocabularies, full and ragged windows, short and long histories.

The history lists are full where a call also applies the update (as they are in a service that has run for
a while with a bounded capacity), so a pass costs the same however many came before it.
"""
import torch

import paper_2512_11280_amd as am

# V = 32000 / 128256 / 152064 are the vocabularies of the package's own workloads; 32003 is not a multiple of a
# vector (most rows then start off a 16-byte boundary); k = 20 is the paper's cap of the window.
LISTED = [
    # a drafted token of one sequence, small vocabulary, float logits: the smallest call there is
    dict(name="draft_one_small", kind="draft", B=1, V=32000, k=4, dtype="f32", idle=0.0),
    # a drafted token of one sequence with a large vocabulary: once per token of a single stream
    dict(name="draft_one", kind="draft", B=1, V=128256, k=8, dtype="bf16", idle=0.0),
    # a drafting call of a batch, some of whose sequences have already stopped drafting
    dict(name="draft_batch", kind="draft", B=32, V=128256, k=8, dtype="bf16", idle=0.25),
    # a drafting call of a full serving batch
    dict(name="draft_large", kind="draft", B=128, V=152064, k=1, dtype="bf16", idle=0.0),
    # entropy and stop flag only (own sampler), float logits
    dict(name="entropy_batch", kind="entropy", B=32, V=128256, k=1, dtype="f32", idle=0.0),
    # one verification round of a single stream: small model, float logits
    dict(name="verify_one_small", kind="verify", B=1, V=32000, k=4, dtype="f32", hist=64, ragged=False, literal=False),
    # one verification round of a single stream, large vocabulary
    dict(name="verify_one", kind="verify", B=1, V=128256, k=8, dtype="bf16", hist=64, ragged=False, literal=False),
    # the ordinary batch: full windows, histories of a thousand distances
    dict(name="verify_batch", kind="verify", B=32, V=128256, k=8, dtype="bf16", hist=1024, ragged=False, literal=False),
    # windows of different lengths, as adaptive drafting makes them, with long histories
    dict(name="verify_ragged", kind="verify", B=64, V=128256, k=16, dtype="bf16", hist=4096, ragged=True, literal=False),
    # the loop exactly as the paper's listing writes it, odd vocabulary; the caller applies the update itself
    dict(name="verify_literal_odd", kind="verify", B=16, V=32003, k=6, dtype="bf16", hist=128, ragged=False, literal=True),
    # float logits (models whose output layer computes in float), the longest window
    dict(name="verify_f32_long", kind="verify", B=8, V=128256, k=20, dtype="f32", hist=256, ragged=False, literal=False),
    # the largest round
    dict(name="verify_large", kind="verify", B=128, V=152064, k=16, dtype="bf16", hist=64, ragged=False, literal=False),
]
_DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}
_SIZE = {"bf16": 2, "f32": 4}
_MOST = 128 * 16 * 152064 * 2 * 2        # bytes of logits of the largest round


def listed():
    return [dict(c) for c in LISTED]


def _log_between(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["verify", "verify", "verify", "draft", "draft", "entropy"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    V = _log_between(rng, 2000, 152064)
    grain = rng.choice([64, 64, 8, 1])   # padded vocabularies mostly, and any size at all
    V = max(V // grain * grain, grain)
    B = _log_between(rng, 1, 128)
    k = rng.randint(1, 20)
    while 2 * B * k * V * _SIZE[dtype] > _MOST:
        B = max(B // 2, 1)
    if kind != "verify":
        return dict(kind=kind, B=B, V=V, k=min(k, 8), dtype=dtype, idle=rng.choice([0.0, 0.25, 0.5]))
    return dict(kind=kind, B=B, V=V, k=k, dtype=dtype, hist=_log_between(rng, 16, 8192),
                ragged=rng.random() < 0.4, literal=rng.random() < 0.25)


def _rows(case, gen):
    """Logits as in the package's workloads: Gaussian target rows with one favoured token, draft rows that mix
    the target row with noise at a weight that differs from sequence to sequence, tokens drawn from the draft."""
    B, k, V, dt = case["B"], case["k"], case["V"], _DTYPE[case["dtype"]]
    dev = "cuda"
    target = torch.empty(B, k + 1, V, dtype=dt, device=dev)
    draft = torch.empty(B, k, V, dtype=dt, device=dev)
    tokens = torch.empty(B, k, dtype=torch.int32, device=dev)
    alpha = 0.5 + 0.48 * torch.rand(B, generator=gen, device=dev)
    spikes = torch.randint(0, V, (B, k + 1, 1), generator=gen, device=dev)
    for b in range(B):
        t = 3.0 * torch.randn(k + 1, V, generator=gen, device=dev)
        t.scatter_add_(1, spikes[b], torch.full((k + 1, 1), 8.0, device=dev))
        d = alpha[b] * t[:k] + (1.0 - alpha[b]) * 3.0 * torch.randn(k, V, generator=gen, device=dev)
        target[b], draft[b] = t, d
        noise = torch.empty(k, V, device=dev).exponential_(generator=gen)
        tokens[b] = (draft[b].float() - noise.log()).argmax(dim=1)
    return target, draft, tokens


def _history(B, n, cap, gen):
    """State of sequences that have decoded for a while: lists of n accepted and n rejected distances around a
    per-sequence threshold."""
    state = am.State(B, cap)
    tau = 0.05 + 0.45 * torch.rand(B, 1, generator=gen, device="cuda")
    for side, lst in ((-0.1, state.LA), (0.1, state.LR)):
        x = tau + side + 0.05 * torch.randn(B, n, generator=gen, device="cuda")
        lst[:, :n] = x.clamp(1e-3, 1 - 1e-3)
    host = state.to_host()
    host["nA"][:] = n
    host["nR"][:] = n
    host["ent_sum"][:] = 4.0 * n
    host["ent_cnt"][:] = n
    host["T_G"][:] = 4.0
    return state.load(host)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, k, V, dt = case["B"], case["k"], case["V"], _DTYPE[case["dtype"]]
    s = dict(kind=case["kind"], seed=seed, round=0)
    if case["kind"] != "verify":
        # the rows of one drafting step inside the round's buffer [B, k, V]
        buf = torch.empty(B, k, V, dtype=dt, device="cuda")
        for b in range(B):
            z = 3.0 * torch.randn(k, V, generator=gen, device="cuda")
            z[:, int(b * 7919 % V)] += 8.0
            buf[b] = z
        active = (torch.rand(B, generator=gen, device="cuda") >= case["idle"]).to(torch.uint8)
        active[0] = 1                    # (a call is only made while some sequence is drafting)
        s.update(rows=buf[:, 0], buf=buf, ws=am.Workspace(B, k, V, dt),
                 T_G=1.0 + 6.0 * torch.rand(B, generator=gen, device="cuda"),
                 active=active,
                 H=torch.empty(B, dtype=torch.float32, device="cuda"),
                 stop=torch.empty(B, dtype=torch.uint8, device="cuda"),
                 token=torch.empty(B, dtype=torch.int32, device="cuda"),
                 status=torch.empty(B, dtype=torch.int32, device="cuda"))
        return s
    target, draft, tokens = _rows(case, gen)
    hist = case["hist"]
    update = not case["literal"]
    s.update(target=target, draft=draft, tokens=tokens, update=update,
             state=_history(B, hist, hist if update else hist + 64, gen),
             lens=torch.randint(1, k + 1, (B,), generator=gen, device="cuda", dtype=torch.int32) if case["ragged"] else None,
             ws=am.Workspace(B, k, V, dt), out=am.binding.alloc_verify_result(B, k),
             options=am.Options(apply_update=1) if update else am.Options(base_test=1, list_update=1))
    return s


def run(s):
    s["round"] += 1
    if s["kind"] == "draft":
        return am.draft_step(s["rows"], s["ws"], T_G=s["T_G"], active=s["active"], step=0, k_max=20, seed=s["seed"],
                             round0=s["round"], H_out=s["H"], stop_out=s["stop"], token_out=s["token"],
                             status_out=s["status"])
    if s["kind"] == "entropy":
        return am.draft_entropy(s["rows"], s["ws"], T_G=s["T_G"], active=s["active"], step=0, k_max=20, H_out=s["H"],
                                stop_out=s["stop"])
    out, st = s["out"], s["state"]
    am.verify(s["target"], s["draft"], s["tokens"], s["ws"], state=st, draft_len=s["lens"], seed=s["seed"],
              round0=s["round"], options=s["options"], out=out)
    r = [out.n_accept, out.next_token, out.H_p, out.H_q, out.d_js, out.p_accept, out.accept_mask, out.status]
    if s["update"]:
        r += [st.T_G, st.ent_sum, st.ent_cnt, st.LA, st.LR, st.nA, st.nR]
    return r


def work(case):
    """Every logit of the positions in the windows once, the lists once, the outputs once (the row that a token is
    drawn from is one of those rows, unless it is a bonus row, which is left out)."""
    B, k, V, es = case["B"], case["k"], case["V"], _SIZE[case["dtype"]]
    if case["kind"] != "verify":
        n = B * (1.0 - case["idle"])
        # per logit: scale and shift, exponential, two accumulations; with the draw two logarithms and a comparison more
        return {"bytes": n * V * es + B * 18.0, "flops": n * V * (11.0 if case["kind"] == "draft" else 6.0)}
    n = B * ((k + 1) / 2.0 if case["ragged"] else k)
    # per pair of logits: two normalisers and entropies (6 each), the distance's term (about 18)
    return {"bytes": 2.0 * n * V * es + 8.0 * B * case["hist"] + 25.0 * B * k,
            "flops": 30.0 * n * V + 8.0 * 2 * n * case["hist"]}


def tolerance(case):
    # Entropies and distances are sums in 32 bits (about 1e-7 apart from one order of summation to another).  The
    # posterior is a ratio of kernel densities whose bandwidth is about 0.02: one part in 1e7 of the distance moves
    # its logarithm by up to 1e-5 where it is far out in a tail.  Whole numbers are the same.
    return {"rel": 1e-5, "max": 2e-4} if case["kind"] == "verify" else {"rel": 2e-6, "max": 1e-5}
