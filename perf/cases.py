"""Performance cases: what a user of this library has it do, with its inputs, its minimum work and its exact results.

A case is a dict of plain values; `kind` names the path.  Every path goes through the binding's calls (the C ABI) in the
order a decode or calibration program makes them, on the default stream, with all buffers owned by the caller.  Inputs
are synthetic, drawn on the GPU from the seed: neuron records N(0, 0.02^2), predictor factors N(0, 1/d) and N(0, 1/r),
hidden states and scores that follow an AR(1) sequence over the tokens, so that consecutive active sets overlap by
80-85% as the method expects.

Kinds:
  decode        T tokens from a cold start: np_predict, np_select_delta, np_stage_gather, np_sparse_mlp per layer
  centroid      the same with centroid prediction: np_centroid_select, np_delta_n, np_stage_gather, np_sparse_mlp_t
                with per-layer counts and thresholds
  predict       np_predict alone (all layers' scores of one token)
  select_delta  T tokens of np_select_delta from a cold start, the scores given
  sparse_mlp    one token's np_sparse_mlp calls, one per layer, every row resident
  dense_mlp     one token's np_dense_mlp calls over the layers of a dense prefix
  calibrate     per-layer thresholds of a token batch (np_act_batch per layer, then np_percentile)
  act_batch     np_act_batch of one layer over a token batch
  stage_rows    np_stage_rows: one token's incoming records from pinned host memory into their slots
"""
import math

import torch

from paper_2608_22643_amd import binding as B
from paper_2608_22643_amd import calibrate
from paper_2608_22643_amd import workload as W

DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}
DEV = "cuda"
WEIGHT_STD = 0.02


def _case(name, kind, layers, d, ffn, dtype, k=1, cap=1, rank=8, act="relu", tokens=1, rho=0.965, **more):
    return dict(name=name, kind=kind, layers=layers, d=d, ffn=ffn, dtype=dtype, k=k, cap=cap, rank=rank, act=act,
                tokens=tokens, rho=rho, **more)


def listed():
    return [
        # the smallest model of the registry: every call is a few microseconds, so launches and latency count
        _case("decode_tiny_f32", "decode", 3, 256, 1024, "f32", 102, 512, 32, tokens=16, rho=0.95),
        # the default configuration of the benchmark: Llama-2-7B-shaped, 15% active, half of the rows resident
        _case("decode_7b_f16", "decode", 31, 4096, 11008, "f16", 1651, 5504, 416, tokens=12),
        # the shape of the paper's evaluated model with its own predictor: centroid heads, SwiGLU, eq. 1 thresholds
        _case("decode_centroid_7b", "centroid", 31, 4096, 14336, "f16", 5500, 7168, 416, act="swiglu", tokens=6,
              rho=0.915, centroids=512, feat=4096),
        # the predictor of the largest configuration: one pass over 4.5 GB of factors per token
        _case("predict_70b_bf16", "predict", 79, 8192, 28672, "bf16", 2867, 10035, 768),
        # selection and delta of a decode at the 7B size: small integer work, once per token, on the critical path
        _case("select_delta_7b", "select_delta", 31, 4096, 11008, "f16", 1651, 5504, tokens=32),
        # the same at the largest size, whose layers are too wide for the 7B kernel
        _case("select_delta_70b", "select_delta", 79, 8192, 28672, "bf16", 2867, 10035, tokens=12, rho=0.977),
        # a small active set (5% of a 7B layer, odd count): the per-call cost of the sparse MLP
        _case("sparse_mlp_7b_5pct", "sparse_mlp", 31, 4096, 11008, "f16", 551, 5504),
        # the largest sparse MLP: 141 MB of records per call, 16 layers
        _case("sparse_mlp_70b_bf16", "sparse_mlp", 16, 8192, 28672, "bf16", 2867, 10035),
        # a dense prefix of eight 7B layers
        _case("dense_mlp_7b_f16", "dense_mlp", 8, 4096, 11008, "f16"),
        # threshold calibration of the whole SwiGLU model on 128 tokens, at the paper's 5,500-row budget
        _case("calibrate_7b_128", "calibrate", 31, 4096, 14336, "f16", 5500, 7168, act="swiglu", tokens=128,
              alpha=61.6),
        # activations of one 13B layer over a longer calibration batch (odd token count)
        _case("act_batch_13b_1999", "act_batch", 1, 5120, 13824, "f16", tokens=1999),
        # the paper's host I/O path: one token's delta (1960 records, 48 MB) from pinned host memory
        _case("stage_rows_7b_host", "stage_rows", 4, 4096, 11008, "f16", 1651, 2752, incoming=490),
    ]


def _log_int(rng, lo, hi, mult=1):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return min(hi, max(lo, v // mult * mult)) if mult > 1 else min(hi, max(lo, v))


def draw(rng):
    """One more case of the listed ranges: the same paths at other widths, counts, types and options."""
    kind = rng.choice(["decode", "centroid", "predict", "select_delta", "sparse_mlp", "dense_mlp", "calibrate",
                       "act_batch"])
    dtype = rng.choice(["f16", "bf16", "f32"])
    act = rng.choice(["relu", "swiglu"])
    mult = 4 if dtype == "f32" else 8
    d = _log_int(rng, 256, 8192, mult)
    ffn = _log_int(rng, 1000, 28672)
    if rng.random() < 0.5:  # real widths are mostly multiples of 16, but any is taken
        ffn = ffn // 16 * 16
    rec = 3 * d * SIZE[dtype]
    c = _case("", kind, 1, d, ffn, dtype, act=act)
    del c["name"]
    cap = min(int(ffn * rng.uniform(0.25, 0.75)), ((1 << 31) - 1) // rec)
    c["cap"] = max(2, cap)
    c["k"] = max(1, min(c["cap"], 8192, int(ffn * math.exp(rng.uniform(math.log(0.05), math.log(0.38))))))
    c["rank"] = _log_int(rng, 32, 512, 8)
    c["rho"] = rng.uniform(0.91, 0.98)
    layers_of = lambda byts, most, hi: max(1, min(hi, int(most / byts)))  # noqa: E731
    if kind in ("decode", "centroid"):
        c["layers"] = rng.randint(1, layers_of((ffn + c["cap"]) * rec, 10e9, 31))
        c["tokens"] = rng.randint(2, 6)
        if kind == "centroid":
            c["centroids"] = _log_int(rng, 32, 512)
            c["feat"] = _log_int(rng, 256, 4096, mult)
    elif kind == "predict":
        c["layers"] = rng.randint(1, layers_of(c["rank"] * (d + ffn) * SIZE[dtype], 4e9, 79))
    elif kind == "select_delta":
        c["layers"] = _log_int(rng, 2, 79)
        c["tokens"] = rng.randint(2, 12)
    elif kind == "sparse_mlp":
        c["layers"] = rng.randint(1, layers_of(c["cap"] * rec, 6e9, 31))
    elif kind == "dense_mlp":
        c["ffn"] = min(ffn, ((1 << 31) - 1) // rec)
        c["k"], c["cap"] = 1, 1
        c["layers"] = rng.randint(1, layers_of(c["ffn"] * rec, 2.5e9, 8))
    else:
        c["ffn"] = min(ffn, 14336, ((1 << 31) - 1) // rec)
        c["d"] = d = min(d, 5120)
        c["k"], c["cap"] = 1, 1
        if kind == "act_batch":
            c["tokens"] = _log_int(rng, 16, 2048)
        else:
            c["tokens"] = _log_int(rng, 16, 256, 4)  # a layer's activations start at a 16-byte boundary
            c["layers"] = rng.randint(1, layers_of(c["ffn"] * rec, 3e9, 31))
            c["alpha"] = round(rng.uniform(40.0, 95.0), 1)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _normal(g, shape, dtype, std=1.0):
    t = torch.empty(shape, dtype=dtype, device=DEV)
    t.normal_(0.0, std, generator=g)
    return t


def _ar1(g, tokens, shape, rho):
    """A list of `tokens` float32 tensors of unit normals, each correlated rho with the one before."""
    out = [_normal(g, shape, torch.float32)]
    for _ in range(1, tokens):
        out.append(_normal(g, shape, torch.float32).mul_(math.sqrt(1.0 - rho * rho)).add_(out[-1], alpha=rho))
    return out


def _i32(*shape):
    return torch.zeros(shape, dtype=torch.int32, device=DEV)


class _State:
    """The buffers of one case, as a program that calls the library keeps them."""


def _lists(c, s):
    """The outputs of the selection and the delta, and the residency state."""
    L, F, k, C = c["layers"], c["ffn"], c["k"], c["cap"]
    s.mask, s.active_ids = _i32(L, (F + 31) // 32), _i32(L, k)
    s.slot_of, s.neuron_of, s.last_used = _i32(L, F), _i32(L, C), _i32(L, F)
    s.state = B.np_state(s.slot_of.data_ptr(), s.neuron_of.data_ptr(), s.last_used.data_ptr())
    s.in_ids, s.in_slots, s.ev_ids, s.ev_slots, s.hit_ids, s.active_slots = (_i32(L, k) for _ in range(6))
    s.counts = _i32(L, 4)
    s.out = B.np_delta_out(*[t.data_ptr() for t in (s.in_ids, s.in_slots, s.ev_ids, s.ev_slots, s.hit_ids,
                                                    s.active_slots, s.counts)])


def _state_outputs(s):
    return {n: getattr(s, n) for n in ("mask", "counts", "slot_of", "neuron_of", "last_used", "active_slots")}


def prepare(case, seed):
    c, s = case, _State()
    s.c = c
    L, d, F, dt, T = c["layers"], c["d"], c["ffn"], DT[c["dtype"]], c["tokens"]
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    kind = c["kind"]
    s.shape = B.make_shape(L, d, F, c["rank"], c["k"], c["cap"], c["dtype"], c["dtype"], c["act"])
    if kind != "act_batch":
        s.ws = torch.zeros(B.np_workspace_size(s.shape), dtype=torch.uint8, device=DEV)
    if kind in ("decode", "predict"):
        s.A = _normal(g, (L, c["rank"], d), dt, 1.0 / math.sqrt(d))
        s.B = _normal(g, (L, F, c["rank"]), dt, 1.0 / math.sqrt(c["rank"]))
    if kind in ("decode", "centroid"):
        s.storage = _normal(g, (L, F, 3 * d), dt, WEIGHT_STD)
        s.resident = torch.zeros((L, c["cap"], 3 * d), dtype=dt, device=DEV)
        s.x = torch.stack(_ar1(g, T, (d,), c["rho"])).to(dt)
        s.y = torch.zeros((T, L, d), dtype=dt, device=DEV)
    if kind in ("decode", "centroid", "select_delta"):
        _lists(c, s)
    if kind == "decode":
        s.scores = [torch.zeros((L, F), dtype=torch.float32, device=DEV) for _ in range(T)]
    elif kind == "centroid":
        K, D = c["centroids"], c["feat"]
        s.heads = _normal(g, (2, L, K, D), dt, 1.0 / math.sqrt(D))
        # the bank: a hot set of each layer's neurons, shared by the two projections, sized so that an intersection
        # holds about 85% of the list capacity k
        hot = min(1.0, max(0.0, (0.85 * c["k"] / F - 0.0025) / (0.6084 - 0.0025)))
        is_hot = torch.rand((L, 1, F), generator=g, device=DEV) < hot
        words = (F + 31) // 32
        s.bank = _i32(2, L, K, words)
        weights = (1 << torch.arange(32, device=DEV, dtype=torch.int64))
        for l in range(L):
            p = torch.where(is_hot[l], 0.78, 0.05)
            for proj in range(2):
                bits = torch.zeros((K, words * 32), dtype=torch.bool, device=DEV)
                bits[:, :F] = torch.rand((K, F), generator=g, device=DEV) < p
                v = (bits.view(K, words, 32).to(torch.int64) * weights).sum(-1)
                s.bank[proj, l] = torch.where(v >= 1 << 31, v - (1 << 32), v).to(torch.int32)
        s.feat = torch.stack(_ar1(g, T, (D,), c["rho"])).to(dt)
        s.model = B.np_centroid_model(K, D, s.heads.data_ptr(), s.bank.data_ptr())
        s.logits = [torch.zeros((2, L, K), dtype=torch.float32, device=DEV) for _ in range(T)]
        s.cids, s.active_counts = _i32(max(2 * L, 4)), _i32(max(L, 4))
        # eq. 1 thresholds near the 61.6th percentile of the activations, one per layer
        z = _normal(g, (2, 20000), torch.float32, WEIGHT_STD * math.sqrt(d))
        a = (torch.nn.functional.silu(z[0]) if c["act"] == "swiglu" else z[0].clamp(min=0)) * z[1]
        t = a.abs().sort().values[12320]
        s.thr = (t * (0.9 + 0.2 * torch.rand(L, generator=g, device=DEV))).float().contiguous()
    elif kind == "predict":
        s.h = _normal(g, (d,), dt)
        s.scores = torch.zeros((L, F), dtype=torch.float32, device=DEV)
    elif kind == "select_delta":
        s.scores = _ar1(g, T, (L, F), c["rho"])
    elif kind == "sparse_mlp":
        s.resident = _normal(g, (L, c["cap"], 3 * d), dt, WEIGHT_STD)
        s.x = _normal(g, (d,), dt)
        s.slots = torch.rand((L, c["cap"]), generator=g, device=DEV).argsort(1)[:, :c["k"]].to(torch.int32).contiguous()
        s.y = torch.zeros((L, d), dtype=dt, device=DEV)
    elif kind == "dense_mlp":
        s.weights = _normal(g, (L, F, 3 * d), dt, WEIGHT_STD)
        s.x = _normal(g, (d,), dt)
        s.y = torch.zeros((L, d), dtype=dt, device=DEV)
    elif kind == "calibrate":
        s.cfg = W.Config("case", L, d, F, c["rank"], 0.1, 0.1, c["dtype"], c["dtype"], T, rho_given=0.0, act=c["act"],
                         k_override=c["k"], c_override=c["cap"])
        s.storage = _normal(g, (L, F, 3 * d), dt, WEIGHT_STD)
        s.x = _normal(g, (T, d), dt)
        s.acts = torch.zeros((L, T, F), dtype=torch.float32, device=DEV)
        s.bytes = s.storage.view(torch.uint8)
        s.flat = s.acts.view(-1)
    elif kind == "act_batch":
        s.weights = _normal(g, (F, 3 * d), dt, WEIGHT_STD)
        s.x = _normal(g, (T, d), dt)
        s.acts = torch.zeros((T, F), dtype=torch.float32, device=DEV)
    elif kind == "stage_rows":
        n, C, k = c["incoming"], c["cap"], c["k"]
        s.host = torch.empty((L, F, 3 * d), dtype=dt, pin_memory=True)
        for l in range(L):
            s.host[l].copy_(_normal(g, (F, 3 * d), dt, WEIGHT_STD))
        s.resident = torch.zeros((L, C, 3 * d), dtype=dt, device=DEV)
        s.plan_counts = torch.zeros((L, 4), dtype=torch.int32, pin_memory=True)
        s.plan_counts[:, 0] = n
        s.plan_ids = torch.zeros((L, k), dtype=torch.int32, pin_memory=True)
        s.plan_slots = torch.zeros((L, k), dtype=torch.int32, pin_memory=True)
        for l in range(L):  # ids and slots ascend, as np_delta gives them
            s.plan_ids[l, :n] = torch.rand(F, generator=g, device=DEV).argsort()[:n].sort().values.int().cpu()
            s.plan_slots[l, :n] = torch.rand(C, generator=g, device=DEV).argsort()[:n].sort().values.int().cpu()
        s.plan = B.np_stage_plan(s.plan_counts.data_ptr(), s.plan_ids.data_ptr(), s.plan_slots.data_ptr())
        s.staging = torch.empty(64 << 20, dtype=torch.uint8, pin_memory=True)
        s.landing = torch.empty(128 << 20, dtype=torch.uint8, device=DEV)
        s.side = torch.cuda.Stream()
        torch.cuda.synchronize()
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s):
    c = s.c
    kind, L, T = c["kind"], c["layers"], c["tokens"]
    if kind == "decode":
        B.np_state_reset(s.shape, s.state, s.ws, None, s.resident)
        for t in range(T):
            x = s.x[t]
            B.np_predict(s.shape, x, s.A, s.B, s.scores[t], s.ws)
            B.np_select_delta(s.shape, t, s.scores[t], s.mask, s.active_ids, s.state, s.out, s.ws)
            B.np_stage_gather(s.shape, s.out, 0, L, s.storage, s.resident, s.ws)
            xp, yp, sp = x.data_ptr(), s.y[t].data_ptr(), s.active_slots.data_ptr()
            for l in range(L):
                B.np_sparse_mlp(s.shape, l, xp, s.resident, sp + l * c["k"] * 4, c["k"],
                                yp + l * c["d"] * SIZE[c["dtype"]], s.ws)
        return {"y": s.y, "scores": s.scores, "active_ids": s.active_ids, **_state_outputs(s)}
    if kind == "centroid":
        B.np_state_reset(s.shape, s.state, s.ws, None, s.resident)
        for t in range(T):
            B.np_centroid_select(s.shape, s.model, s.feat[t], s.logits[t], s.cids, s.mask, s.active_ids,
                                 s.active_counts, s.ws)
            B.np_delta_n(s.shape, t, s.active_ids, s.active_counts, s.state, s.out, s.ws)
            B.np_stage_gather(s.shape, s.out, 0, L, s.storage, s.resident, s.ws)
            xp, yp, sp = s.x[t].data_ptr(), s.y[t].data_ptr(), s.active_slots.data_ptr()
            for l in range(L):
                B.np_sparse_mlp_t(s.shape, l, xp, s.resident, sp + l * c["k"] * 4, c["k"], s.active_counts, s.thr,
                                  yp + l * c["d"] * SIZE[c["dtype"]], s.ws)
        return {"y": s.y, "logits": s.logits, "cids": s.cids[:2 * L], "active_counts": s.active_counts[:L],
                **_state_outputs(s)}
    if kind == "predict":
        B.np_predict(s.shape, s.h, s.A, s.B, s.scores, s.ws)
        return s.scores
    if kind == "select_delta":
        B.np_state_reset(s.shape, s.state, s.ws, None)
        for t in range(T):
            B.np_select_delta(s.shape, t, s.scores[t], s.mask, s.active_ids, s.state, s.out, s.ws)
        return {"active_ids": s.active_ids, "in_ids": s.in_ids, "in_slots": s.in_slots, "ev_ids": s.ev_ids,
                "ev_slots": s.ev_slots, "hit_ids": s.hit_ids, **_state_outputs(s)}
    if kind == "sparse_mlp":
        yp, sp = s.y.data_ptr(), s.slots.data_ptr()
        for l in range(L):
            B.np_sparse_mlp(s.shape, l, s.x, s.resident, sp + l * c["k"] * 4, c["k"],
                            yp + l * c["d"] * SIZE[c["dtype"]], s.ws)
        return s.y
    if kind == "dense_mlp":
        yp, wp, row = s.y.data_ptr(), s.weights.data_ptr(), c["d"] * SIZE[c["dtype"]]
        for l in range(L):
            B.np_dense_mlp(s.shape, wp + l * c["ffn"] * 3 * row, s.x, yp + l * row, s.ws)
        return s.y
    if kind == "calibrate":
        thr = calibrate.thresholds(s.cfg, s.bytes, s.x, T, c["alpha"], s.ws, None, s.flat)
        return {"thresholds": thr, "acts": s.acts}
    if kind == "act_batch":
        B.np_act_batch(s.shape, s.weights, s.x, T, s.acts)
        return s.acts
    B.np_stage_rows(s.shape, s.plan, 0, L, s.host, s.resident, s.staging, s.staging.numel(), s.landing,
                    s.landing.numel(), s.side)
    return s.resident.view(torch.int32)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    c = case
    L, d, F, T, k, r, w = c["layers"], c["d"], c["ffn"], c["tokens"], c["k"], c["rank"], SIZE[c["dtype"]]
    rec, kind = 3 * d * w, c["kind"]
    # selection and delta: scores, slot_of and last_used read, the lists and the state of the active rows written
    sd = T * L * (3 * 4 * F + 4 * c["cap"] + 10 * 4 * k)
    # rows staged: the first token's whole set, then what the resident buffer misses (about a tenth of the set)
    staged = L * k * (1 + 0.1 * (T - 1))
    if kind == "decode":
        return {"bytes": T * (L * r * (d + F) * w + L * k * rec + L * F * 4 + L * d * w) + 2 * staged * rec + sd,
                "flops": 2 * T * (L * r * (d + F) + 3 * L * k * d)}
    if kind == "centroid":
        act = 0.85 * k
        heads = 2 * L * c["centroids"] * c["feat"]
        return {"bytes": T * (heads * w + L * act * rec + L * d * w) + 2 * 0.85 * staged * rec + sd,
                "flops": 2 * T * (heads + 3 * L * act * d)}
    if kind == "predict":
        return {"bytes": L * r * (d + F) * w + L * F * 4, "flops": 2 * L * r * (d + F)}
    if kind == "select_delta":
        return {"bytes": sd, "flops": 0}
    if kind == "sparse_mlp":
        return {"bytes": L * (k * rec + 4 * k + 2 * d * w), "flops": 6 * L * k * d}
    if kind == "dense_mlp":
        return {"bytes": L * (F * rec + 2 * d * w), "flops": 6 * L * F * d}
    if kind == "calibrate":
        return {"bytes": L * (2 * F * d * w + 2 * T * F * 4) + T * d * w, "flops": 4 * L * T * F * d}
    if kind == "act_batch":
        return {"bytes": 2 * F * d * w + T * d * w + T * F * 4, "flops": 4 * T * F * d}
    return {"bytes": 2 * L * c["incoming"] * rec, "flops": 0}


# ---------------------------------------------------------------------------
# results
# ---------------------------------------------------------------------------

def tolerance(case):
    """Selection, delta and staged bytes have one correct value.  Floating outputs: fp32 sums of the same products in
    another order (measured against 64 bits: 2e-7 for scores, 6e-7 for activations), the MLP's rounded once to the
    output type (measured 2.1e-4 in f16, 1.7e-3 in bf16)."""
    kind, dtype = case["kind"], case["dtype"]
    if kind in ("select_delta", "stage_rows"):
        return "exact"
    mlp = {"f32": {"rel": 2e-6, "max": 2e-5}, "f16": {"rel": 4e-4, "max": 4e-3}, "bf16": {"rel": 3e-3, "max": 4e-2}}
    if kind in ("sparse_mlp", "dense_mlp"):
        return mlp[dtype]
    if kind == "decode":  # near-ties of two orderings may exchange a neuron, which moves a few list entries
        return dict(mlp[dtype], differ=0.01)
    if kind == "centroid":  # an activation within rounding of its threshold may go either way: one row of y
        return {"rel": 3e-3 if dtype == "bf16" else 1.5e-3, "max": 6e-2, "differ": 0.01}
    return {"rel": 2.5e-6, "max": 2.5e-5}


def _act(c, gate, up):
    return (gate / (1 + torch.exp(-gate)) if c["act"] == "swiglu" else gate.clamp(min=0)) * up


def _mlp64(c, rec, x, thr=None):
    """The gated MLP over the records `rec` [n][3d], in 64 bits."""
    d, r, x = c["d"], rec.double(), x.double()
    a = _act(c, r[:, :d] @ x, r[:, d:2 * d] @ x)
    if thr is not None:
        a = torch.where(a.abs() < float(thr), torch.zeros_like(a), a)
    return a @ r[:, 2 * d:]


def exact(case, seed):
    c = case
    kind, L, T, d, k = c["kind"], c["layers"], c["tokens"], c["d"], c["k"]
    if kind in ("select_delta", "stage_rows"):
        return None
    s = prepare(case, seed)
    if kind == "predict":
        return torch.stack([s.B[l].double() @ (s.A[l].double() @ s.h.double()) for l in range(L)])
    if kind == "decode":
        y = torch.zeros((T, L, d), dtype=torch.float64, device=DEV)
        scores = torch.zeros((T, L, c["ffn"]), dtype=torch.float64, device=DEV)
        for l in range(L):
            scores[:, l] = (s.x.double() @ s.A[l].double().t()) @ s.B[l].double().t()
            for t in range(T):
                y[t, l] = _mlp64(c, s.storage[l][scores[t, l].topk(k).indices], s.x[t])
        return {"y": y, "scores": list(scores)}
    if kind == "centroid":
        y = torch.zeros((T, L, d), dtype=torch.float64, device=DEV)
        logits = torch.zeros((T, 2, L, c["centroids"]), dtype=torch.float64, device=DEV)
        bit = torch.arange(32, device=DEV)
        for l in range(L):
            for proj in range(2):
                logits[:, proj, l] = s.feat.double() @ s.heads[proj, l].double().t()
            for t in range(T):
                word = s.bank[0, l, logits[t, 0, l].argmax()] & s.bank[1, l, logits[t, 1, l].argmax()]
                ids = ((word[:, None] >> bit) & 1).reshape(-1)[:c["ffn"]].nonzero()[:k, 0]
                y[t, l] = _mlp64(c, s.storage[l][ids], s.x[t], s.thr[l])
        return {"y": y, "logits": list(logits)}
    if kind == "sparse_mlp":
        return torch.stack([_mlp64(c, s.resident[l][s.slots[l].long()], s.x) for l in range(L)])
    if kind == "dense_mlp":
        return torch.stack([_mlp64(c, s.weights[l], s.x) for l in range(L)])
    acts = lambda w: _act(c, s.x.double() @ w[:, :d].double().t(), s.x.double() @ w[:, d:2 * d].double().t())  # noqa: E731
    if kind == "act_batch":
        return acts(s.weights)
    m = min(max(math.ceil(c["alpha"] * T * c["ffn"] / 100.0), 1), T * c["ffn"])
    out, thr = torch.zeros((L, T, c["ffn"]), dtype=torch.float64, device=DEV), []
    for l in range(L):
        out[l] = acts(s.storage[l])
        thr.append(out[l].abs().flatten().sort().values[m - 1])
    return {"thresholds": torch.stack(thr), "acts": out}
