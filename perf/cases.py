"""The calls this library is measured on, through its public entry points.

The library is the hot path of an overlapped training or serving step on one
GPU: bf16 GEMMs with the weight stored K x N (``occ_gemm``) or N x K
(``occ_gemm_bt``), the local share of an allreduce (``share_reduce``,
``share_reduce_own``) or of an alltoall (``share_permute``), and the two-stream
schedule of both (``occ_overlap_enqueue``).  ``listed`` names fixed cases,
``draw`` gives others of the same ranges; ``prepare`` makes what a program holds
before the call, ``run`` is the call.
"""
import math

import torch

from paper_2606_09200_amd import binding as occ
from paper_2606_09200_amd import inputs

DEV = "cuda:0"
MIB = 1 << 20


def listed():
    return [
        # the smallest GEMM of the repository's workloads: launch and latency
        dict(name="gemm_512", op="gemm", layout="kn", M=512, N=512, K=512),
        # a small batch through a projection with a long inner dimension: few output tiles
        dict(name="gemm_1k_longk", op="gemm", layout="nk", M=1024, N=1024, K=4096),
        # an ordinary layer of a mid-size model
        dict(name="gemm_2k", op="gemm", layout="kn", M=2048, N=2048, K=4096),
        # the compute-bound GEMM every overlap measurement is quoted on
        dict(name="gemm_8k", op="gemm", layout="kn", M=8192, N=8192, K=8192),
        # an expert's linear layer over a long sequence, weight as stored by a linear layer
        dict(name="gemm_expert", op="gemm", layout="nk", M=16384, N=14336, K=4096),
        # a ragged number of tokens against an odd-sized output (a vocabulary shard)
        dict(name="gemm_ragged", op="gemm", layout="nk", M=3001, N=5003, K=2504),
        # one decode step of 16 sequences: the weight is read once
        dict(name="gemm_decode", op="gemm", layout="kn", M=16, N=28672, K=8192, std_b=0.02),
        # a decode step of a larger batch (or a very short prefill)
        dict(name="gemm_batch", op="gemm", layout="nk", M=64, N=28672, K=8192, std_b=0.02),
        # the allreduce share paired with the compute-bound GEMM
        dict(name="reduce_8", op="reduce", nchunks=8, length=1 << 25),
        # a gradient bucket of an odd number of elements from 6 ranks, held as one (6, length) buffer
        dict(name="reduce_ragged", op="reduce", nchunks=6, length=11000003),
        # the alltoall share of the expert layer
        dict(name="permute_64", op="permute", nchunks=64, chunk_bytes=4 * MIB),
        # the schedule itself: each iteration's allreduce share consumes its GEMM's output
        dict(name="overlap_own", op="overlap", comm="own", layout="kn", M=8192, N=8192, K=8192, nchunks=7,
             n_iter=4, lds_bytes=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, mult=1):
    """A size of [lo, hi] spread over its logarithm: half of them round, half any multiple of `mult`."""
    x = _log(rng, lo, hi)
    step = max(mult, 128) if x >= 256 and rng.random() < 0.5 else mult
    return max(mult, min(hi, (x + step // 2) // step * step))


def _draw_gemm(rng):
    layout = rng.choice(("kn", "nk"))
    kind = rng.choice(("decode", "batch", "square", "square"))
    nmult = 8 if layout == "kn" else 1
    if kind == "decode":
        M = rng.randint(1, 16)
        N, K = _size(rng, 1024, 28672, nmult), _size(rng, 512, 8192, 8)
    elif kind == "batch":
        M = _size(rng, 17, 512)
        N, K = _size(rng, 1024, 28672, nmult), _size(rng, 512, 8192, 8)
    else:
        M, N, K = _size(rng, 128, 8192), _size(rng, 128, 8192, nmult), _size(rng, 128, 8192, 8)
    return dict(op="gemm", layout=layout, M=M, N=N, K=K, std_b=1.0 if kind == "square" else 0.02)


def draw(rng):
    op = rng.choice(("gemm", "gemm", "gemm", "reduce", "own", "permute", "overlap"))
    if op == "gemm":
        return _draw_gemm(rng)
    if op in ("reduce", "own"):
        n = rng.choice((2, 3, 4, 5, 6, 7, 8, 8, 12, 16))
        length = _size(rng, 1 << 16, (1 << 28) // n)
        return dict(op=op, nchunks=n if op == "reduce" else n - 1, length=length)
    if op == "permute":
        n = rng.choice((4, 7, 8, 16, 31, 32, 64, 128, 256))
        # tokens of whole 16-byte rows, or of an odd number of 16-bit values
        mult = 16 if rng.random() < 0.67 else 2
        return dict(op=op, nchunks=n, chunk_bytes=_size(rng, 4096, 256 * MIB // n, mult))
    comm = rng.choice(("own", "reduce", "permute"))
    layout = rng.choice(("kn", "nk"))
    M, N, K = (_size(rng, 512, 4096, 8) for _ in range(3))
    case = dict(op="overlap", comm=comm, layout=layout, M=M, N=N, K=K, n_iter=rng.randint(2, 8),
                lds_bytes=rng.choice((0, 0, 16 << 10)))
    if comm == "own":
        case["nchunks"] = rng.choice((1, 3, 7))
    elif comm == "reduce":
        case.update(nchunks=rng.choice((2, 4, 8)), length=_size(rng, 1 << 18, 1 << 24))
    else:
        case.update(nchunks=rng.choice((8, 16, 64)), chunk_bytes=_size(rng, 1 << 16, 4 * MIB, 16))
    return case


_comm_stream = None


def _comm():
    """The program's one communication stream (default priority)."""
    global _comm_stream
    if _comm_stream is None:
        _comm_stream = torch.cuda.Stream(device=DEV)
    return _comm_stream


def _operands(case, seed):
    A, Bt = inputs.gemm_operands(case["M"], case["N"], case["K"], seed=seed, std_b=case.get("std_b", 1.0),
                                 device=DEV)
    return A, (Bt.t().contiguous() if case["layout"] == "kn" else Bt)


def _collective(case, seed):
    """The collective's inputs and its output buffer."""
    kind = case.get("comm", case["op"])
    if kind == "permute":
        n, cb = case["nchunks"], case["chunk_bytes"]
        return dict(src=inputs.permute_payload(n, cb, seed=seed, device=DEV),
                    perm=inputs.chunk_permutation(n, seed=seed), chunk_bytes=cb,
                    dst=torch.empty(n * cb, dtype=torch.uint8, device=DEV))
    length = case["M"] * case["N"] if case["op"] == "overlap" and kind == "own" else case["length"]
    return dict(bufs=inputs.reduce_chunks(case["nchunks"], length, seed=seed, device=DEV),
                out=torch.empty(length, device=DEV))


def _own(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randn(case["length"], generator=g, device=DEV, dtype=torch.float32).to(torch.bfloat16)


def prepare(case, seed):
    s = dict(case)
    op = case["op"]
    if op == "gemm":
        s["A"], s["B"] = _operands(case, seed)
        s["C"] = torch.empty((case["M"], case["N"]), device=DEV, dtype=torch.bfloat16)
        return s
    s["coll"] = _collective(case, seed + 1)
    if op == "own":
        s["own"] = _own(case, seed + 2)
    if op == "overlap":
        s["A"], s["B"] = _operands(case, seed)
        shape = (case["M"], case["N"])
        if case["comm"] == "own":
            shape = (case["n_iter"],) + shape
        s["C"] = torch.empty(shape, device=DEV, dtype=torch.bfloat16)
        s["workspace"] = torch.zeros(occ.occ_overlap_workspace_bytes(case["n_iter"]), dtype=torch.uint8, device=DEV)
        s["comm_stream"] = _comm()
    return s


def run(s):
    op = s["op"]
    if op == "gemm":
        return (occ.occ_gemm if s["layout"] == "kn" else occ.occ_gemm_bt)(s["A"], s["B"], s["C"])
    c = s["coll"]
    if op == "reduce":
        return occ.share_reduce(c["bufs"], c["out"])
    if op == "own":
        return occ.share_reduce_own(s["own"], c["bufs"], c["out"])
    if op == "permute":
        return occ.share_permute(c["src"], c["dst"], c["perm"], c["chunk_bytes"])
    comp, comm = torch.cuda.current_stream(), s["comm_stream"]
    comm.wait_stream(comp)
    occ.occ_overlap_enqueue(s["A"], s["B"], s["C"], workspace=s["workspace"], comm_stream=comm,
                            lds_bytes=s["lds_bytes"], n_iter=s["n_iter"], b_layout=s["layout"],
                            reduce_own=s["comm"] == "own", **c)
    comp.wait_stream(comm)
    return {"C": s["C"], "out": c["dst"] if s["comm"] == "permute" else c["out"]}


def _gemm_work(case):
    M, N, K = case["M"], case["N"], case["K"]
    return 2.0 * (M * K + K * N), 2.0 * M * N, 2.0 * M * N * K  # bytes in, bytes out, flops


def work(case):
    op = case["op"]
    if op == "gemm":
        i, o, f = _gemm_work(case)
        return {"bytes": i + o, "flops": f}
    kind = case.get("comm", op)
    if kind == "permute":
        cin = cout = float(case["nchunks"] * case["chunk_bytes"])
        adds = 0.0
    else:
        length = case["M"] * case["N"] if op == "overlap" and kind == "own" else case["length"]
        cin, cout = 4.0 * length * case["nchunks"], 4.0 * length
        adds = float(length) * (case["nchunks"] - (0 if kind == "own" else 1))
        if op == "own":
            cin += 2.0 * length
    if op != "overlap":
        return {"bytes": cin + cout, "flops": adds}
    # each iteration runs its GEMM and its collective; with "own" the collective reads the GEMM's output back
    i, o, f = _gemm_work(case)
    n = case["n_iter"]
    return {"bytes": n * (i + o + cin + cout + (o if kind == "own" else 0.0)), "flops": n * (f + adds)}


def tolerance(case):
    # the chunk sums are defined bit for bit (binary32, left to right) and the permutation copies bytes
    if case["op"] in ("reduce", "own", "permute"):
        return "exact"
    # bf16 outputs of fp32 sums: one rounding is 1.7e-3 of the result in the 2-norm and at most 2^-8 of a value
    return {"rel": 7e-3, "max": 1.6e-2}


def exact(case, seed):
    s = prepare(case, seed)
    op = s["op"]
    if op in ("gemm", "overlap"):
        A, B = s["A"].double(), s["B"].double()
        C = A @ (B if s["layout"] == "kn" else B.t())
        if op == "gemm":
            return C
    c = s["coll"]
    if case.get("comm", op) == "permute":
        n = case["nchunks"]
        out = c["src"].view(n, -1)[c["perm"].long().to(DEV)].reshape(-1)
    else:
        if op == "own":
            out, first = s["own"].double(), 0
        elif op == "overlap" and case["comm"] == "own":
            out, first = C.reshape(-1).clone(), 0
        else:
            out, first = c["bufs"][0].double(), 1
        for b in c["bufs"][first:]:
            out += b
    if op != "overlap":
        return out
    return {"C": C.expand(s["C"].shape) if case["comm"] == "own" else C, "out": out}
