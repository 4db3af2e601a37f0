"""The calls this library is used for, as cases that can be prepared, run, checked and timed.

A case is a dict of plain values:

  name       (listed cases only)
  entry      which calls one pass makes: "reduce" (dart_reduce), "static" (dart_reduce_static),
             "norms" (dart_reduce_with_norms), "stages" (the four stage entry points one after
             the other), "sequences" (dart_reduce on spans, then dart_compact_sequences)
  data       how the hidden states are distributed: "clusters", "copies", "video", "audio"
  dtype      "bf16" or "f32"
  B, n_lo, n_hi, ragged, len_seed
             samples and their tokens; dense: n_lo == n_hi; ragged: lengths drawn from
             [n_lo, n_hi] with len_seed (the first two samples have the two extremes)
  D, P       hidden size, pivots per sample
  P_ext      pivots of the P that are rows from outside the samples (text tokens)
  K          tokens kept per sample, or 0: floor(N * keep_num / keep_den)
  crit_D     width of a separate criterion tensor (key states), 0: the hidden states themselves
  pivots     "max_l1", "min_l1" or "random"
  rule       "per_pivot", "min" or "max" (the retention rule)

The inputs are made on the GPU from the seed alone; the sizes come from the case alone.
"""
import math
import random

import torch

import paper_2502_11494_amd as dart

DTYPES = {"bf16": (torch.bfloat16, dart.DART_BF16, 2), "f32": (torch.float32, dart.DART_F32, 4)}
PIVOTS = {"max_l1": dart.DART_PIVOT_MAX_L1, "min_l1": dart.DART_PIVOT_MIN_L1,
          "random": dart.DART_PIVOT_RANDOM}
RULES = {"per_pivot": dart.DART_SCORE_PER_PIVOT, "min": dart.DART_SCORE_MIN,
         "max": dart.DART_SCORE_MAX}
N_KV, KV_WIDTH = 4, 1024  # cached key / value tensors moved along by the "sequences" entry
NORMS_ERR = 1e-5  # relative error the caller's norms are declared with ("norms" entry)


def _case(**kw):
    base = dict(entry="reduce", data="clusters", dtype="bf16", B=1, n_lo=576, n_hi=576,
                ragged=False, len_seed=0, D=4096, P=8, P_ext=0, K=0, keep_num=111, keep_den=1000,
                crit_D=0, pivots="max_l1", rule="per_pivot")
    base.update(kw)
    return base


def listed():
    return [
        # one camera frame of a robot policy, 256 tokens kept down to 56, in a control loop that
        # cannot allocate: the smallest call, all latency and launches
        _case(name="action_frame", entry="static", B=1, n_lo=256, n_hi=256, K=56),
        # one 576-token image held in fp32
        _case(name="image_f32", dtype="f32", B=1, K=64),
        # a serving batch of 576-token images
        _case(name="images", B=16, K=128),
        # the pivot ablation's text tokens: 4 visual and 4 text pivots, hidden size of a 13B model
        _case(name="text_pivots", B=16, D=5120, P=8, P_ext=4, K=128),
        # utterances of different lengths, packed, most tokens kept
        _case(name="audio", data="audio", B=16, n_lo=300, n_hi=1500, ragged=True, len_seed=5,
              D=3072, P=8, keep_num=700),
        # high-resolution multi-crop images with exact copies: the headline batch
        _case(name="multicrop", data="copies", B=8, n_lo=2880, n_hi=2880, P=16, K=320),
        # the same batch with the criterion norms handed over by the key projection's epilogue
        _case(name="multicrop_norms", entry="norms", data="copies", B=8, n_lo=2880, n_hi=2880,
              P=16, K=320, crit_D=1024),
        # one threshold for all pivots, hidden size of a 72B model
        _case(name="one_threshold", B=8, D=8192, P=8, K=192, rule="min"),
        # the stage entry points on their own, fp32, an odd number of tokens
        _case(name="stages_f32", entry="stages", dtype="f32", B=4, n_lo=1445, n_hi=1445, D=2048,
              P=16, K=161),
        # vision spans inside whole sequences: hidden states, cached key / value rows and three
        # planes of position ids shrink together
        _case(name="sequences", entry="sequences", B=8, n_lo=700, n_hi=3600, ragged=True,
              len_seed=9, D=3584, P=16, keep_num=222),
        # video frames: near duplicates everywhere, many pivots
        _case(name="video", data="video", B=4, n_lo=9216, n_hi=9216, D=3584, P=32, K=1024),
        # dynamic-resolution images, packed: the largest call
        _case(name="ragged", B=32, n_lo=1024, n_hi=16384, ragged=True, len_seed=3, D=3584, P=16),
    ]


def _between(rng, lo, hi):
    """A whole number in [lo, hi], spread over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A case of the same ranges: any entry, any size up to a third of the largest listed one."""
    while True:
        c = _case()
        c["entry"] = rng.choice(["reduce", "reduce", "reduce", "static", "norms", "stages",
                                 "sequences"])
        c["dtype"] = rng.choice(["bf16", "bf16", "bf16", "f32"])
        c["data"] = rng.choice(["clusters", "copies", "video", "audio"])
        c["D"] = rng.choice([1024, 1536, 2048, 2560, 3072, 3584, 4096, 5120, 8192,
                             8 * rng.randint(120, 640)])
        c["P"] = rng.choice([4, 8, 8, 16, 16, 32, rng.randint(1, 40)])
        c["ragged"] = c["entry"] == "sequences" or rng.random() < 0.4
        c["len_seed"] = rng.randint(0, 999)
        c["B"] = _between(rng, 1, 32)
        top = _between(rng, 200, 12000 if c["dtype"] == "bf16" else 3000)
        c["n_hi"] = top
        c["n_lo"] = rng.randint(max(100, top // 4), top) if c["ragged"] else top
        c["keep_num"] = rng.choice([111, 111, 222, 333, 500, 700, rng.randint(60, 800)])
        if not c["ragged"]:
            c["K"] = c["n_lo"] * c["keep_num"] // 1000
        kept = c["n_lo"] * c["keep_num"] // 1000
        if rng.random() < 0.2:
            c["P_ext"] = c["P"] // 2
        what = rng.random()
        if what < 0.12:
            c["pivots"] = "min_l1"
        elif what < 0.22 and c["entry"] in ("reduce", "static"):
            c["pivots"] = "random"
        if c["pivots"] != "random" and rng.random() < 0.3:
            c["crit_D"] = rng.choice([256, 512, 1024, 8 * rng.randint(30, 130)])
        if c["entry"] != "stages" and rng.random() < 0.15:
            c["rule"] = rng.choice(["min", "max"])
        rows, esz = sum(_lengths(c)), DTYPES[c["dtype"]][2]
        size = rows * c["D"] * esz
        if kept < c["P"] or size > (560 << 20) or (c["dtype"] == "f32" and size > (128 << 20)):
            continue
        if c["entry"] == "static":  # what the built-in scratch buffer holds
            if rows * (12 * c["P"] + 28) + c["B"] * 800 + 4096 > (24 << 20):
                continue
        return c


# ---- sizes ---------------------------------------------------------------------------------

def _lengths(case):
    if not case["ragged"]:
        return [case["n_lo"]] * case["B"]
    r = random.Random(case["len_seed"])
    n = [r.randint(case["n_lo"], case["n_hi"]) for _ in range(case["B"])]
    n[0] = case["n_hi"]
    if len(n) > 1:
        n[1] = case["n_lo"]
    return n


def _budgets(case):
    return [case["K"] if case["K"] > 0 else n * case["keep_num"] // case["keep_den"]
            for n in _lengths(case)]


def _text_rows(case):
    """Rows of text before and after the span of every sequence."""
    r = random.Random(case["len_seed"] + 1)
    return [(r.randint(30, 40), r.randint(20, 60)) for _ in range(case["B"])]


def work(case):
    """One read of every input and one write of every output; the products of the scores."""
    esz = DTYPES[case["dtype"]][2]
    rows, kept = sum(_lengths(case)), sum(_budgets(case))
    D, P = case["D"], case["P"]
    nbytes = rows * D * esz + rows * case["crit_D"] * esz + case["B"] * case["P_ext"] * D * esz
    if case["entry"] == "norms":
        # the criterion rows themselves are not needed, their norms are
        nbytes += 4 * rows - rows * case["crit_D"] * esz
    if case["entry"] == "sequences":
        moved = kept + sum(a + b for a, b in _text_rows(case))
        nbytes += (moved - kept) * D * esz             # text rows read
        nbytes += moved * D * esz + 2 * N_KV * moved * KV_WIDTH * esz + 2 * 3 * 8 * moved
        nbytes += 4 * kept
    else:
        nbytes += kept * (D * esz + 8 + 8 + 4)         # rows, position ids (both ways), indices
    if case["entry"] == "stages":
        nbytes += 4 * rows * P                         # the scores are an output
    return {"bytes": nbytes, "flops": 2 * rows * D * (P + 1)}


def tolerance(case):
    """Retained sets, rows, position ids and offsets are exact.  The stage entry points also
    return the scores and the norms as fp32: against 64 bits the scores show up to 2e-8 and the
    norms, sums of up to 8192 terms in fp32, up to 4.5e-8 over ninety drawn cases."""
    if case["entry"] == "stages":
        return {"rel": 2e-7, "max": 4e-6, "differ": 0.0}
    return "exact"


# ---- inputs --------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _tokens(g, case, n):
    """Hidden states of one sample, fp32 [n, D]: near-duplicate tokens abound, as they do after
    an early decoder layer."""
    D = case["D"]
    if case["data"] == "video":  # 144 tokens per frame, every frame the last one plus drift
        per = min(144, n)
        cent = _randn(g, 16, D)
        x = cent[torch.randint(0, 16, (per,), generator=g, device="cuda")] + 0.1 * _randn(g, per, D)
        frames = -(-n // per)
        drift = 0.02 * _randn(g, frames, per, D)
        drift[0] = x
        return torch.cumsum(drift, 0).reshape(frames * per, D)[:n]
    if case["data"] == "audio":  # runs of 3..12 frames share a centroid
        cent = _randn(g, 64, D)
        runs = torch.randint(3, 13, (n // 3 + 1,), generator=g, device="cuda")
        which = torch.randint(0, 64, (n // 3 + 1,), generator=g, device="cuda")
        which = torch.repeat_interleave(which, runs)[:n]
        return cent[which] + 0.1 * _randn(g, n, D)
    groups = max(16, min(256, n // 8)) if case["data"] == "copies" else max(16, n // 16)
    cent = _randn(g, groups, D)
    x = cent[torch.randint(0, groups, (n,), generator=g, device="cuda")] + 0.1 * _randn(g, n, D)
    if case["data"] == "copies":  # a tenth of the tokens are bit-exact copies of others
        perm = torch.randperm(n, generator=g, device="cuda")
        m = n // 10
        src = perm[m:][torch.randint(0, n - m, (m,), generator=g, device="cuda")]
        x[perm[:m]] = x[src]
    return x


def _inputs(case, seed):
    """Everything a user's program holds: the same tensors for prepare() and exact()."""
    g = _generator(seed)
    dt = DTYPES[case["dtype"]][0]
    lens = _lengths(case)
    rows, D = sum(lens), case["D"]
    text = _text_rows(case) if case["entry"] == "sequences" else [(0, 0)] * len(lens)
    x_rows = rows + sum(a + b for a, b in text)
    s = dict(lens=lens, budgets=_budgets(case), text=text)
    X = torch.empty((x_rows, D), dtype=dt, device="cuda")
    starts, at = [], 0
    for n, (a, b) in zip(lens, text):
        if a + b:
            X[at:at + a] = _randn(g, a, D).to(dt)
            X[at + a + n:at + a + n + b] = _randn(g, b, D).to(dt)
        X[at + a:at + a + n] = _tokens(g, case, n).to(dt)
        starts.append(at + a)
        at += a + n + b
    s["X"], s["starts"] = X, starts
    s["crit"] = None
    if case["crit_D"] > 0:  # key rows: a few tokens of massive norm
        c = _randn(g, x_rows, case["crit_D"])
        heavy = torch.rand((x_rows, 1), generator=g, device="cuda") < 0.02
        scale = 1.5 + 2.5 * torch.rand((x_rows, 1), generator=g, device="cuda")
        s["crit"] = (c * torch.where(heavy, scale, torch.ones_like(scale))).to(dt)
    s["ext"] = None
    if case["P_ext"] > 0:  # text rows, each blended with a token of its sample
        e = _randn(g, case["B"], case["P_ext"], D)
        for b, (n, r0) in enumerate(zip(lens, starts)):
            pick = torch.randint(0, n, (case["P_ext"],), generator=g, device="cuda")
            e[b] = 0.5 * e[b] + 0.5 * X[r0 + pick].float()
        s["ext"] = e.reshape(-1, D).to(dt)
    s["draw_seed"] = int(seed)
    if case["entry"] == "sequences":
        s["kv"] = [_randn(g, x_rows, KV_WIDTH).to(dt) for _ in range(N_KV)]
        s["pos"] = torch.arange(3 * x_rows, dtype=torch.int64, device="cuda").reshape(3, x_rows)
    else:
        s["pos"] = torch.cat([torch.arange(n, dtype=torch.int64, device="cuda") for n in lens])
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    dt, code, _ = DTYPES[case["dtype"]]
    lens, rows, kept = s["lens"], sum(s["lens"]), sum(s["budgets"])
    B, D, P, x_rows = case["B"], case["D"], case["P"], s["X"].shape[0]
    s["entry"] = case["entry"]
    more = dict(pivot_mode=PIVOTS[case["pivots"]], score_mode=RULES[case["rule"]],
                ext_pivots=s["ext"], P_ext=case["P_ext"], seed=s["draw_seed"], K=case["K"],
                keep_num=case["keep_num"], keep_den=case["keep_den"])
    if case["ragged"]:
        cu = [0]
        for n in lens:
            cu.append(cu[-1] + n)
        s["cu"] = torch.tensor(cu, dtype=torch.int32, device="cuda")
        more.update(cu_seqlens=s["cu"], total_N=rows, max_N=max(lens))
    else:
        more.update(N=lens[0])
    if case["entry"] == "sequences":
        seq = [0]
        for n, (a, b) in zip(lens, s["text"]):
            seq.append(seq[-1] + a + n + b)
        s["seq_cu"] = torch.tensor(seq, dtype=torch.int32, device="cuda")
        s["span"] = torch.tensor(s["starts"], dtype=torch.int32, device="cuda")
        more.update(span_start=s["span"], X_rows=x_rows)
    s["desc"] = dart.make_desc(B, D, P, code, **more)
    s["ws"] = None if case["entry"] == "static" else dart.alloc_workspace(s["desc"])
    s["crit_kw"] = {}
    if s["crit"] is not None:
        s["crit_kw"] = dict(crit=s["crit"], crit_D=case["crit_D"], crit_ld=case["crit_D"])
    if case["entry"] == "norms":
        s["l1"] = (s["X"] if s["crit"] is None else s["crit"]).float().abs().sum(1)
    new = lambda shape, dtype: torch.empty(shape, dtype=dtype, device="cuda")  # noqa: E731
    s["keep"] = new(kept, torch.int32)
    s["cu_keep"] = new(B + 1, torch.int32)
    if case["entry"] == "sequences":
        out_rows = x_rows - rows + kept
        s["pairs"] = [(t, new((out_rows, t.shape[1]), dt)) for t in [s["X"]] + s["kv"]]
        s["row_map"] = new(out_rows, torch.int32)
        s["seq_cu_out"] = new(B + 1, torch.int32)
        s["pos_out"] = new((3, out_rows), torch.int64)
    else:
        s["Y"] = new((kept, D), dt)
        s["pos_out"] = new(kept, torch.int64)
    if case["entry"] == "stages":
        s["piv"] = new(B * P, torch.int32)
        s["l1"] = new(rows, torch.float32)
        s["S"] = new(rows * P, torch.float32)
    return s


# ---- one pass ------------------------------------------------------------------------------

def run(s):
    d, X, ws = s["desc"], s["X"], s["ws"]
    if s["entry"] == "stages":
        dart.dart_select_pivots(d, X, s["piv"], ws, l1_out=s["l1"], **s["crit_kw"])
        dart.dart_duplication_scores(d, X, s["piv"], s["S"], ws)
        dart.dart_topk_keep(d, s["S"], s["piv"], s["keep"], ws, X=X, cu_keep=s["cu_keep"])
        dart.dart_gather_compact(d, X, s["keep"], s["Y"], ws, pos=s["pos"], pos_out=s["pos_out"])
        return {k: s[k] for k in ("Y", "pos_out", "keep", "cu_keep", "piv", "S", "l1")}
    if s["entry"] == "sequences":
        dart.dart_reduce(d, X, None, s["keep"], ws, cu_keep=s["cu_keep"], **s["crit_kw"])
        dart.dart_compact_sequences(d, s["seq_cu"], s["keep"], s["pairs"], s["seq_cu_out"],
                                    s["row_map"], ws, pos=s["pos"], pos_out=s["pos_out"])
        return {"rows": [dst for _, dst in s["pairs"]], "pos_out": s["pos_out"],
                "row_map": s["row_map"], "seq_cu_out": s["seq_cu_out"], "keep": s["keep"],
                "cu_keep": s["cu_keep"]}
    kw = dict(pos=s["pos"], pos_out=s["pos_out"], cu_keep=s["cu_keep"], **s["crit_kw"])
    if s["entry"] == "static":
        dart.dart_reduce_static(d, X, s["Y"], s["keep"], **kw)
    elif s["entry"] == "norms":
        dart.dart_reduce_with_norms(d, X, s["Y"], s["keep"], ws, s["l1"], NORMS_ERR, **kw)
    else:
        dart.dart_reduce(d, X, s["Y"], s["keep"], ws, **kw)
    return {k: s[k] for k in ("Y", "pos_out", "keep", "cu_keep")}


# ---- the same in 64 bits -------------------------------------------------------------------

def _philox(counter, key):
    """Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11)."""
    c, k, m32 = list(counter), list(key), 0xFFFFFFFF
    for r in range(10):
        if r:
            k = [(k[0] + 0x9E3779B9) & m32, (k[1] + 0xBB67AE85) & m32]
        p0, p1 = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]
        c = [(p1 >> 32) ^ c[1] ^ k[0], p1 & m32, (p0 >> 32) ^ c[3] ^ k[1], p0 & m32]
    return c


def _drawn(seed, b, n, count):
    got, t = [], 0
    while len(got) < count:
        w = _philox((t // 4, b, 0, 0), (seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF))[t % 4]
        d = (w * n) >> 32
        if d not in got:
            got.append(d)
        t += 1
    return got


def _norms64(rows):
    return torch.cat([r.double().abs().sum(1) for r in rows.split(4096)])


def _reduce64(case, s, b):
    """Pivots, norms, scores and retained tokens of sample b.  Every score is a sum over its own
    row, so that equal rows tie exactly; ties go to the lowest index."""
    n, k, r0 = s["lens"][b], s["budgets"][b], s["starts"][b]
    P, P_in = case["P"], case["P"] - case["P_ext"]
    X = s["X"][r0:r0 + n]
    l1 = _norms64((s["X"] if s["crit"] is None else s["crit"])[r0:r0 + n])
    if case["pivots"] == "random":
        tokens = _drawn(s["draw_seed"], b, n, P_in)
    else:
        order = torch.argsort(l1, descending=case["pivots"] == "max_l1", stable=True)
        tokens = order[:P_in].tolist()
    ext = s["ext"][b * case["P_ext"]:(b + 1) * case["P_ext"]] if case["P_ext"] else X[:0]
    pivot_rows = torch.cat([X[tokens], ext]).double()
    S = torch.empty((P, n), dtype=torch.float64, device=X.device)
    for j in range(0, n, 4096):
        x = X[j:j + 4096].double()
        xn = x.square().sum(1).sqrt()
        for i in range(P):
            S[i, j:j + 4096] = (x * pivot_rows[i]).sum(1) / (xn * pivot_rows[i].square().sum().sqrt())
    kept = torch.zeros(n, dtype=torch.bool, device=X.device)
    kept[tokens] = True
    spare = k - P_in
    if case["rule"] == "per_pivot":
        for i in range(P):
            q = spare // P + (1 if i < spare % P else 0)
            row = torch.where(kept, torch.full_like(S[i], float("inf")), S[i])
            kept[torch.argsort(row, stable=True)[:q]] = True
    else:
        row = S.amin(0) if case["rule"] == "min" else S.amax(0)
        row = torch.where(kept, torch.full_like(row, float("inf")), row)
        kept[torch.argsort(row, stable=True)[:spare]] = True
    piv = torch.tensor(tokens + [-1 - e for e in range(case["P_ext"])], dtype=torch.int32,
                       device=X.device)
    return piv, l1, S, torch.nonzero(kept).flatten()


def exact(case, seed):
    s = _inputs(case, seed)
    piv, l1, S, keep, rows, cu_keep = [], [], [], [], [], [0]
    for b in range(case["B"]):
        p, l, sc, k = _reduce64(case, s, b)
        piv.append(p)
        l1.append(l)
        S.append(sc.flatten())
        keep.append(k.int())
        rows.append(s["starts"][b] + k)
        cu_keep.append(cu_keep[-1] + len(k))
    out = {"keep": torch.cat(keep), "cu_keep": torch.tensor(cu_keep, dtype=torch.int32)}
    if case["entry"] == "sequences":
        row_map, seq, at = [], [0], 0
        for b, (n, (a, t)) in enumerate(zip(s["lens"], s["text"])):
            every = torch.arange(at, at + a + n + t, device="cuda")
            row_map.append(torch.cat([every[:a], rows[b], every[a + n:]]))
            seq.append(seq[-1] + len(row_map[-1]))
            at += a + n + t
        row_map = torch.cat(row_map)
        out.update(rows=[t[row_map].double() for t in [s["X"]] + s["kv"]],
                   pos_out=s["pos"][:, row_map], row_map=row_map.int(),
                   seq_cu_out=torch.tensor(seq, dtype=torch.int32))
        return out
    rows = torch.cat(rows)
    out.update(Y=s["X"][rows].double(), pos_out=s["pos"][rows])
    if case["entry"] == "stages":
        out.update(piv=torch.cat(piv), S=torch.cat(S), l1=torch.cat(l1))
    return out
