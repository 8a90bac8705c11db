"""The work that is timed: the calls a training program makes through the package's public entry points.

Kinds of case, one per entry point of the hot path:
  reduce   lagom_comm_kernel, reduce-copy: one local reduction step of a collective
  gather   lagom_comm_kernel, gather-copy: one all-gather (or all-to-all) share
  ring     lagom_comm_steps: one rank's share of a ring all-reduce, P-1 reduce and P-1 copy steps in one launch
  gemm     lagom_gemm, both weight layouts, bf16 and fp32 results
  layers   a training step's overlapped part: all-gathers on one stream, the GEMMs that use the gathered weights on
           another, GEMM i waiting for all-gather i-1
  profile  lagom_overlap_run: one measured co-run, which the parameter search makes at every step it takes

Communication parameters (channels, threads, chunk bytes) are an input of every communication, as they are for a user:
the collective library's default (8, 256, 2 MiB), what the search picks on the workloads' grids (up to 32 channels), and
the wide launches used when nothing runs beside them.
"""
import math

import torch

from paper_2602_20656_amd import binding as lg

KiB, MiB = 1 << 10, 1 << 20
DT = {"f32": (lg.LAGOM_F32, torch.float32, 4), "bf16": (lg.LAGOM_BF16, torch.bfloat16, 2)}


def listed():
    return [
        # two peers' fp32 gradients of 2^20 elements added on four channels: the smallest reduce of the workloads
        {"name": "reduce_pair_f32", "kind": "reduce", "dtype": "f32", "nsrc": 2, "ndst": 1, "count": 1 << 20,
         "nc": 4, "nt": 256, "chunk": 128 * KiB},
        # reduce-scatter share of a 4096 x 8192 activation over eight ranks, nothing beside it: wide launch
        {"name": "reduce_tp_wide", "kind": "reduce", "dtype": "bf16", "nsrc": 8, "ndst": 1, "count": 4194304,
         "nc": 256, "nt": 512, "chunk": 32 * KiB},
        # sixteen ranks, a length that no vector width divides, on the channels left beside a computation
        {"name": "reduce_16_ragged", "kind": "reduce", "dtype": "bf16", "nsrc": 16, "ndst": 1, "count": 1000003,
         "nc": 32, "nt": 256, "chunk": 64 * KiB},
        # all-gather of eight 4 MiB weight shards with the collective library's default parameters
        {"name": "gather_default", "kind": "gather", "dtype": "bf16", "nsrc": 8, "ndst": 1, "count": 2097152,
         "nc": 8, "nt": 256, "chunk": 2 * MiB},
        # shards of odd length: every shard but the first starts off a 16-byte boundary in the destination
        {"name": "gather_ragged", "kind": "gather", "dtype": "bf16", "nsrc": 8, "ndst": 1, "count": 1000003,
         "nc": 32, "nt": 256, "chunk": 64 * KiB},
        # ring all-reduce share of a 25 MiB gradient bucket over eight ranks, searched parameters
        {"name": "ring_bucket", "kind": "ring", "dtype": "bf16", "ranks": 8, "count": 1638400,
         "nc": 32, "nt": 256, "chunk": 64 * KiB},
        # the smallest product of the workloads
        {"name": "gemm_512", "kind": "gemm", "m": 512, "n": 512, "k": 512, "b_is_nk": True, "out": "bf16"},
        # few rows against a long reduction: a short micro-batch through a projection
        {"name": "gemm_few_rows", "kind": "gemm", "m": 33, "n": 1000, "k": 4096, "b_is_nk": True, "out": "bf16"},
        # a data-gradient product (weight read as [K,N], fp32 result) with no size a multiple of the tile
        {"name": "gemm_ragged_grad", "kind": "gemm", "m": 4100, "n": 4200, "k": 2056, "b_is_nk": False, "out": "f32"},
        # the largest product of the workloads
        {"name": "gemm_8192", "kind": "gemm", "m": 8192, "n": 8192, "k": 8192, "b_is_nk": True, "out": "bf16"},
        # eight FSDP layers: the next layer's weight is gathered while this layer multiplies
        {"name": "layers_fsdp", "kind": "layers", "pairs": 8, "m": 8192, "n": 4096, "k": 4096, "ranks": 8,
         "nc": 32, "nt": 256, "chunk": 32 * KiB},
        # one profile of the gradient-bucket group: the ring share beside a 4096^3 product, 5 timed repetitions
        {"name": "profile_bucket", "kind": "profile", "dtype": "bf16", "ranks": 8, "count": 1638400,
         "m": 4096, "n": 4096, "k": 4096, "iters": 5, "nc": 32, "nt": 256, "chunk": 64 * KiB},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _with_cfg(rng, case):
    """Adds communication parameters; few light channels are given to small buffers only (about a millisecond at most)."""
    nc, nt = rng.choice((4, 8, 16, 32, 64, 128, 256)), rng.choice((128, 256, 512, 1024))
    while work(case)["bytes"] > 200 * KiB * nc * nt:
        nc *= 2
    return {**case, "nc": nc, "nt": nt, "chunk": rng.choice((16, 32, 64, 128, 256, 512, 1024, 2048)) * KiB}


def draw(rng):
    """One more case: sizes log-uniform over the range between the smallest and the largest listed ones."""
    kind = rng.choice(("reduce", "reduce", "gather", "gather", "ring", "gemm", "gemm", "gemm", "gemm", "layers", "profile"))
    if kind == "reduce":
        return _with_cfg(rng, {"kind": kind, "dtype": rng.choice(("f32", "bf16")), "nsrc": rng.randint(2, 16),
                               "ndst": rng.choice((1, 1, 2)), "count": _log(rng, 1 << 16, 1 << 22)})
    if kind == "gather":
        count = _log(rng, 1 << 16, 1 << 21)
        return _with_cfg(rng, {"kind": kind, "dtype": rng.choice(("f32", "bf16")), "nsrc": rng.randint(2, 16),
                               "ndst": rng.choice((1, 1, 2)), "count": rng.choice((count, count // 8 * 8))})
    if kind == "ring":
        return _with_cfg(rng, {"kind": kind, "dtype": rng.choice(("f32", "bf16")), "ranks": rng.choice((2, 4, 8, 16)),
                               "count": _log(rng, 1 << 15, 1 << 21) // 8 * 8})
    if kind == "gemm":
        nk = rng.random() < 0.5
        m, n, k = _log(rng, 32, 8192), _log(rng, 64, 8192), _log(rng, 64, 8192) // 8 * 8
        if rng.random() < 0.5:      # as often a multiple of 128, as model widths are
            m, n, k = max(128, m // 128 * 128), max(128, n // 128 * 128), max(128, k // 128 * 128)
        return {"kind": kind, "m": m, "n": n if nk else max(8, n // 8 * 8), "k": k, "b_is_nk": nk, "out": rng.choice(("bf16", "bf16", "f32"))}
    m, n, k = (_log(rng, 1024, 4096) // 128 * 128 for _ in range(3))
    cfg = {"nc": rng.choice((8, 16, 32, 64)), "nt": rng.choice((128, 256)), "chunk": rng.choice((32, 64, 128)) * KiB}
    if kind == "layers":
        return {"kind": kind, "pairs": rng.randint(2, 6), "m": m, "n": n, "k": k, "ranks": rng.choice((4, 8)), **cfg}
    return {"kind": kind, "dtype": "bf16", "ranks": rng.choice((4, 8)), "count": _log(rng, 1 << 17, 1 << 20) // 8 * 8,
            "m": m, "n": n, "k": k, "iters": rng.randint(3, 8), **cfg}


# ------------------------------------------------------------------------------------------------ inputs
_STREAMS = []


def _streams():
    """A pair of streams whose kernels overlap, drawn once, as a program does at its start."""
    if not _STREAMS:
        _STREAMS.extend(lg.overlapping_streams())
    return _STREAMS


def _values(gen, shape, dtype, scale=1.0, uniform=False):
    """Gradients, activations and weights are normal at the scale of their use; the fp32 reduces take U[-1, 1)."""
    x = torch.empty(shape, dtype=torch.float32, device="cuda")
    x = x.uniform_(-1.0, 1.0, generator=gen) if uniform else x.normal_(0.0, scale, generator=gen)
    return x.to(dtype)


def _ring(gen, case):
    """Rank 0's buffers and the steps of its share: P-1 times out = incoming + local (the last one also stored
    locally), then P-1 times store and forward; two wire buffers each way."""
    _, dtype, esz = DT[case["dtype"]]
    P, m = case["ranks"], case["count"]
    local = _values(gen, P * m, dtype, 0.125)
    wire_in = [_values(gen, m, dtype, 0.125) for _ in range(2)]
    wire_out = [torch.zeros(m, dtype=dtype, device="cuda") for _ in range(2)]
    chunk = [local.data_ptr() + c * m * esz for c in range(P)]
    steps = []
    for s in range(P - 1):
        c = (-s - 1) % P
        steps.append((lg.LAGOM_REDUCE_COPY, [wire_in[s % 2], chunk[c]], [wire_out[s % 2]] + ([chunk[c]] if s == P - 2 else [])))
    for s in range(P - 1):
        steps.append((lg.LAGOM_GATHER_COPY, [wire_in[s % 2]], [chunk[-s % P]] + ([wire_out[s % 2]] if s < P - 2 else [])))
    return local, wire_in, wire_out, steps


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    kind = case["kind"]
    s = {"case": case, "kind": kind}
    if "nc" in case:
        s["cfg"] = (case["nc"], case["nt"], case["chunk"])
    if kind in ("reduce", "gather"):
        _, dtype, _ = DT[case["dtype"]]
        s["srcs"] = [_values(gen, case["count"], dtype, uniform=case["dtype"] == "f32") for _ in range(case["nsrc"])]
        n = case["count"] * (case["nsrc"] if kind == "gather" else 1)
        s["dsts"] = [torch.zeros(n, dtype=dtype, device="cuda") for _ in range(case["ndst"])]
    if kind in ("ring", "profile"):
        s["local"], s["wire_in"], s["wire_out"], s["steps"] = _ring(gen, case)
    if kind in ("gemm", "profile"):
        m, n, k = case["m"], case["n"], case["k"]
        nk = case.get("b_is_nk", True)
        s["A"] = _values(gen, (m, k), torch.bfloat16)
        s["B"] = _values(gen, (n, k) if nk else (k, n), torch.bfloat16, 0.02)
        s["C"] = torch.zeros((m, n), dtype=DT[case.get("out", "bf16")][1], device="cuda")
    if kind == "layers":
        m, n, k, P = case["m"], case["n"], case["k"], case["ranks"]
        s["A"] = _values(gen, (m, k), torch.bfloat16)
        s["first"] = _values(gen, (n, k), torch.bfloat16, 0.02)           # the first layer's weight is there already
        s["shards"] = [[_values(gen, n * k // P, torch.bfloat16, 0.02) for _ in range(P)] for _ in range(case["pairs"])]
        s["weights"] = [torch.zeros((n, k), dtype=torch.bfloat16, device="cuda") for _ in range(case["pairs"])]
        s["C"] = [torch.zeros((m, n), dtype=torch.bfloat16, device="cuda") for _ in range(case["pairs"])]
        s["streams"] = _streams()
        s["gathered"] = [torch.cuda.Event() for _ in range(case["pairs"])]
    if kind == "profile":
        s["streams"] = _streams()
        s["launches"] = [lg.CommLaunch(op, DT[case["dtype"]][0], srcs, dsts, case["count"], 0, fuse=i > 0)
                         for i, (op, srcs, dsts) in enumerate(s["steps"])]
        s["comps"] = [lg.GemmDesc(s["A"], s["B"], s["C"], case["m"], case["n"], case["k"])]
        torch.cuda.synchronize()       # inputs come from torch's stream, the runner has its own two
    return s


def run(s):
    case, kind = s["case"], s["kind"]
    if kind in ("reduce", "gather"):
        lg.lagom_comm_kernel(lg.LAGOM_REDUCE_COPY if kind == "reduce" else lg.LAGOM_GATHER_COPY, DT[case["dtype"]][0],
                             s["srcs"], s["dsts"], case["count"], s["cfg"], torch.cuda.current_stream())
        return s["dsts"]
    if kind == "ring":
        lg.lagom_comm_steps(DT[case["dtype"]][0], s["steps"], case["count"], s["cfg"], torch.cuda.current_stream())
        return [s["local"]] + s["wire_out"]
    if kind == "gemm":
        lg.lagom_gemm(s["A"], s["B"], s["C"], case["m"], case["n"], case["k"], case["b_is_nk"], DT[case["out"]][0],
                      torch.cuda.current_stream())
        return s["C"]
    if kind == "layers":
        main, (s_comm, s_comp) = torch.cuda.current_stream(), s["streams"]
        s_comm.wait_stream(main)
        s_comp.wait_stream(main)
        n_shard = case["n"] * case["k"] // case["ranks"]
        for i in range(case["pairs"]):
            lg.lagom_comm_kernel(lg.LAGOM_GATHER_COPY, lg.LAGOM_BF16, s["shards"][i], [s["weights"][i]], n_shard, s["cfg"], s_comm)
            s["gathered"][i].record(s_comm)
            if i > 0:
                s_comp.wait_event(s["gathered"][i - 1])
            lg.lagom_gemm(s["A"], s["weights"][i - 1] if i > 0 else s["first"], s["C"][i], case["m"], case["n"], case["k"],
                          True, lg.LAGOM_BF16, s_comp)
        main.wait_stream(s_comm)
        main.wait_stream(s_comp)
        return s["weights"] + s["C"]
    lg.lagom_overlap_run(s["launches"], [s["cfg"]], s["comps"], *s["streams"], 1, case["iters"], lg.LAGOM_CORUN)
    return [s["local"]] + s["wire_out"] + [s["C"]]


# ------------------------------------------------------------------------------------------------ what a pass costs
def _ring_work(case):
    """Each step reads its sources and writes its destinations (a ring's steps are dictated by the wire)."""
    esz, P, m = DT[case["dtype"]][2], case["ranks"], case["count"]
    moved = (P - 1) * 3 + 1 + (P - 1) * 3 - 1        # (2 read, 1 or 2 written), then (1 read, 2 or 1 written)
    return {"bytes": moved * m * esz, "flops": (P - 1) * m}


def _gemm_work(case):
    m, n, k = case["m"], case["n"], case["k"]
    return {"bytes": 2 * (m * k + n * k) + m * n * DT[case.get("out", "bf16")][2], "flops": 2 * m * n * k}


def work(case):
    kind = case["kind"]
    if kind == "reduce":
        return {"bytes": lg.lagom_comm_bytes(lg.LAGOM_REDUCE_COPY, DT[case["dtype"]][0], case["nsrc"], case["ndst"], case["count"]),
                "flops": (case["nsrc"] - 1) * case["count"]}
    if kind == "gather":
        return {"bytes": lg.lagom_comm_bytes(lg.LAGOM_GATHER_COPY, DT[case["dtype"]][0], case["nsrc"], case["ndst"], case["count"]), "flops": 0}
    if kind == "ring":
        return _ring_work(case)
    if kind == "gemm":
        return _gemm_work(case)
    if kind == "layers":
        g, gathered = _gemm_work(case), 4 * case["n"] * case["k"]
        return {"bytes": case["pairs"] * (g["bytes"] + gathered), "flops": case["pairs"] * g["flops"]}
    r, g, reps = _ring_work(case), _gemm_work(case), 1 + case["iters"]
    return {"bytes": reps * (r["bytes"] + g["bytes"]), "flops": reps * (r["flops"] + g["flops"])}


def tolerance(case):
    """Communication is exact: the order of the additions and the rounding are part of its definition.  Products: fp32
    sums in another order, measured against torch's fp32 product of the same inputs (K 512 to 8192).  fp32 results differ
    by rel 1.1e-6, max 8e-6; bf16 results by rel 7e-5, from values that round to the neighbouring bf16 (at most 2^-7
    of the value)."""
    if case["kind"] in ("reduce", "gather", "ring"):
        return "exact"
    if case.get("out") == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 3e-4, "max": 1.6e-2}
