"""The calls by which the speed of this library is judged: absorbed-MLA decode attention through the Python entry
points of `paper_2509_25224_amd.amla`, on what a serving program holds in device memory at that point -- the step's
query rows, the paged latent cache, the block table, the lengths.

A case says how many sequences the step has (`batch`), how many new tokens each (`s_q`), how many heads this GPU holds
(`heads`; 128 is the whole model, fewer one GPU's slice of it under tensor parallelism), how long the cached prefixes
are (`lo` .. `hi`, drawn once per case from `lengths_seed`), how wide the block table is (`table_blocks`, 0: just the
longest sequence's), which rescale and which options the program selected, and how wide the logits are (`q_sigma`)."""
import torch

from paper_2509_25224_amd import accounting, amla, workloads

SCALE = workloads.SOFTMAX_SCALE
BLOCK = workloads.BLOCK
VARIANT = {"add": amla.AMLA_RESCALE_ADD, "mul": amla.AMLA_RESCALE_MUL, "add_comp": amla.AMLA_RESCALE_ADD_COMP}
FLAGS = {"": 0, "balanced": amla.AMLA_FLAG_BALANCED, "causal": amla.AMLA_FLAG_CAUSAL,
         "iteration_512": amla.AMLA_FLAG_ITERATION_512}
# the most cached tokens (times query rows, and alone) of a drawn case: those of the largest listed one
MOST_ROW_KEYS = 8 * 65536 * 4 * 128
MOST_KEYS = 256 * 4096


def _case(name, batch, s_q, heads, lo, hi, lengths_seed=0, table_blocks=0, variant="add", flags="", q_lens=False,
          static=False, q_sigma=1.0):
    return {"name": name, "batch": batch, "s_q": s_q, "heads": heads, "lo": lo, "hi": hi, "lengths_seed": lengths_seed,
            "table_blocks": table_blocks, "variant": variant, "flags": flags, "q_lens": q_lens, "static": static,
            "q_sigma": q_sigma}


def listed():
    return [
        # the smallest call: one short sequence on one GPU of an eight-way tensor-parallel group (configuration 0)
        _case("tiny_h16", 1, 1, 16, 256, 256),
        # one user, all heads, a prompt of odd length, a block table laid out for 16384 tokens
        _case("single_user", 1, 1, 128, 3001, 3001, table_blocks=256),
        # a lightly loaded server, one GPU's slice of the heads, short ragged prompts
        _case("light_load_h32", 6, 1, 32, 100, 1500, lengths_seed=11),
        # two drafted tokens per sequence, few sequences, through the entry point that allocates nothing
        _case("draft_b12_static", 12, 2, 128, 700, 2100, lengths_seed=12, variant="mul", static=True),
        # ordinary decode: one token of 64 sequences (configuration 1)
        _case("decode_b64", 64, 1, 128, 4096, 4096),
        # the paper's Table 5 shape at 2048 keys, with the compensated rescale
        _case("table5_b96_comp", 96, 1, 128, 2048, 2048, variant="add_comp"),
        # multi-token prediction, two tokens of 128 sequences (configuration 2, what bench.py times)
        _case("mtp_b128", 128, 2, 128, 4096, 4096),
        # ragged continuous batching, library's own decomposition (configuration 3)
        _case("ragged_b32", 32, 2, 128, 1024, 16384, lengths_seed=3),
        # the same batch from a program that asks for the balanced decomposition
        _case("ragged_b32_balanced", 32, 2, 128, 1024, 16384, lengths_seed=3, flags="balanced"),
        # speculative decoding: up to three tokens, as many as each sequence has, masked among themselves
        _case("speculative_b40", 40, 3, 128, 130, 5000, lengths_seed=13, flags="causal", q_lens=True),
        # long context, four tokens, wide logits (configuration 4)
        _case("long_b8", 8, 4, 128, 65536, 65536, q_sigma=4.0),
        # one GPU's sixteen heads over a large batch: bound by reading the cache
        _case("shard_h16_b256", 256, 1, 16, 4096, 4096),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    heads = rng.choice((128, 128, 128, 64, 32, 16, log_int(1, 128)))
    s_q = rng.choice((1, 1, 2, 2, 3, 4))
    hi = log_int(40, 65536)
    lo = hi if rng.random() < 0.4 else max(1, int(hi * rng.uniform(0.05, 0.9)))
    most = min(MOST_ROW_KEYS // (hi * s_q * heads), MOST_KEYS // hi, 256)
    batch = log_int(1, max(1, most))
    flags = rng.choice(("", "", "", "", "balanced", "causal", "iteration_512"))
    variant = rng.choice(("add", "add", "mul", "add" if flags == "iteration_512" else "add_comp"))
    blocks = (hi + BLOCK - 1) // BLOCK
    case = _case("", batch, s_q, heads, lo, hi, lengths_seed=rng.randrange(1 << 20),
                 table_blocks=blocks + rng.randrange(blocks + 1) if rng.random() < 0.4 else 0, variant=variant, flags=flags,
                 q_lens=flags == "causal" and rng.random() < 0.5, static=rng.random() < 0.15,
                 q_sigma=rng.choice((1.0, 1.0, 2.0, 4.0)))
    del case["name"]
    if case["static"] and amla.amla_workspace_bytes(_desc(case)) > amla.amla_static_workspace_limit() // 2:
        case["static"] = False
    return case


def _lengths(case):
    return workloads.ragged_lengths(case["lengths_seed"], case["batch"], case["lo"], case["hi"])


def _tokens(case):
    """New tokens of each sequence."""
    if case["q_lens"]:
        return workloads.ragged_lengths(case["lengths_seed"] + 1, case["batch"], 1, case["s_q"])
    return workloads.ragged_lengths(0, case["batch"], case["s_q"], case["s_q"])


def _keys_seen(case):
    """(sequence, token, number of keys it attends to) of every new token."""
    for b, (n, tokens) in enumerate(zip(_lengths(case).tolist(), _tokens(case).tolist())):
        for t in range(tokens):
            yield b, t, max(0, n - (tokens - 1 - t)) if case["flags"] == "causal" else n


def _table_blocks(case):
    return max(case["table_blocks"], -(-int(_lengths(case).max()) // BLOCK))


def _pool_blocks(case):
    need = int(((_lengths(case) + BLOCK - 1) // BLOCK).sum())
    return need + need // 8 + 1   # some of the pool is always free


def _desc(case):
    return amla.make_desc(case["batch"], case["s_q"], case["heads"], _pool_blocks(case), _table_blocks(case),
                          VARIANT[case["variant"]], 0, FLAGS[case["flags"]])


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(seed)
    batch, s_q, heads = case["batch"], case["s_q"], case["heads"]
    lengths = _lengths(case)

    def normal(*shape):
        t = torch.empty(shape, dtype=torch.bfloat16, device=dev)
        for part in t.split(max(1, (1 << 26) // (t.numel() // shape[0]))):
            part.copy_(torch.randn(part.shape, generator=gen, device=dev))
        return t

    q = normal(batch, s_q, heads, workloads.D_QK)
    q *= case["q_sigma"]
    kv = normal(_pool_blocks(case), BLOCK, workloads.D_QK)
    # the pool's blocks in random order, dealt to the sequences; -1 where a sequence has no block
    order = torch.randperm(_pool_blocks(case), generator=gen, device=dev).to(torch.int32).cpu()
    table = torch.full((batch, _table_blocks(case)), -1, dtype=torch.int32)
    at = 0
    for b, n in enumerate(lengths):
        blocks = -(-int(n) // BLOCK)
        table[b, :blocks] = order[at:at + blocks]
        at += blocks
    state = {"q": q, "kv": kv, "table": table.to(dev), "lengths": torch.from_numpy(lengths).to(dev), "static": case["static"],
             "options": {"variant": VARIANT[case["variant"]], "flags": FLAGS[case["flags"]]}}
    if case["q_lens"]:
        state["options"]["q_lens"] = torch.from_numpy(_tokens(case)).to(dev)
    if case["static"]:
        state["out"] = torch.empty((batch, s_q, heads, workloads.D_V), dtype=torch.bfloat16, device=dev)
        state["lse"] = torch.empty((batch, s_q, heads), dtype=torch.float32, device=dev)
    return state


def run(state):
    args = (state["q"], state["kv"], state["table"], state["lengths"], SCALE)
    if state["static"]:
        return amla.amla_decode_static_workspace(*args, state["out"], state["lse"], **state["options"])
    return amla.amla_decode(*args, **state["options"])


def work(case):
    total, batch = int(_lengths(case).sum()), case["batch"]
    padding = case["heads"] * (batch * case["s_q"] - int(_tokens(case).sum()))   # query rows that nobody has to read
    small = 4 * batch * (1 + case["q_lens"]) + 4 * int(-(-_lengths(case) // BLOCK).sum())   # lengths, counts, block numbers
    return {"bytes": accounting.algorithmic_bytes(case["heads"], case["s_q"], batch, total) - padding * 2 * workloads.D_QK + small,
            "flops": accounting.decode_flops(case["heads"], 1, sum(seen for _, _, seen in _keys_seen(case)))}


def tolerance(case):
    # The weights and the output are rounded to bf16: the relative error against 64 bits is 1.5e-3 .. 2.1e-3 over these
    # ranges (the largest single difference 1.8e-2), and two implementations that split the keys elsewhere differ by as much.
    return {"rel": 8e-3, "max": 0.07}


def exact(case, seed):
    """softmax(scale q K^T) V in float64, one sequence at a time."""
    state = prepare(case, seed)
    q, kv, table = state["q"], state["kv"], state["table"]
    batch, s_q, heads = case["batch"], case["s_q"], case["heads"]
    out = torch.zeros((batch, s_q, heads, workloads.D_V), dtype=torch.float64, device=q.device)
    lse = torch.full((batch, s_q, heads), -float("inf"), dtype=torch.float64, device=q.device)
    for b, t, seen in _keys_seen(case):
        if seen > 0:
            keys = kv[table[b, :-(-seen // BLOCK)].long()].reshape(-1, workloads.D_QK)[:seen].double()
            logits = (q[b, t].double() @ keys.t()) * SCALE
            lse[b, t] = torch.logsumexp(logits, dim=1)
            out[b, t] = torch.softmax(logits, dim=1) @ keys[:, :workloads.D_V]
    return out, lse
