"""Workloads of the sparse product C = A x B as a program that serves or evaluates pruned layers meets
them: fp32, A given once in CSR and turned into a plan, B and C dense on the GPU, through
`plan_create` and `Plan.execute`.

Shapes, sparsities, row-length laws and widths are those of this repository's configurations (the tiny,
convolution, feed-forward, stress and sweep matrices of workloads/generators.py) and of its benchmark and
tests (narrow B of 4 to 16 columns, ragged sizes, 200 columns without a hint).  A case is

  rows, cols   M and K of A
  sparsity     share of A that is pruned (the mean over the rows)
  law          how the entries that are kept spread over the rows: "magnitude" (global magnitude pruning of
               normal weights: even rows), "lognormal" (feed-forward layers: row densities of sigma 0.5) or
               "zipf" (few rows hold most entries, one row in twenty is empty)
  width        N, the columns of B and C
  hint         the plan is created with n_hint = width (False: without a hint)
  keep_out     the program keeps C and hands it in (False: execute allocates it)
  new_plan     the pass includes the creation of the plan from host CSR arrays
"""
import math

import numpy as np
import torch

import paper_2506_15174_amd as spmm


def _case(name, rows, cols, sparsity, law, width, hint=True, keep_out=False, new_plan=False):
    return dict(name=name, rows=rows, cols=cols, sparsity=sparsity, law=law, width=width, hint=hint,
                keep_out=keep_out, new_plan=new_plan)


def listed():
    return [
        # the smallest configuration: a call is launch latency and host work
        _case("tiny", 256, 256, 0.90, "magnitude", 32),
        # a 1x1-convolution layer, output buffer kept by the program
        _case("conv", 512, 2048, 0.80, "magnitude", 128, keep_out=True),
        # the two feed-forward projections of a Transformer block, uneven row densities
        _case("ffn_up", 4096, 1024, 0.70, "lognormal", 128),
        _case("ffn_down", 1024, 4096, 0.90, "lognormal", 64),
        # token-by-token decoding: a handful of columns
        _case("decode_4", 4096, 4096, 0.80, "magnitude", 4, keep_out=True),
        _case("decode_16", 2048, 8192, 0.70, "magnitude", 16),
        # highly pruned square layers, ordinary and narrow batches
        _case("sparse_95", 4096, 4096, 0.95, "magnitude", 128),
        _case("sparse_98", 8192, 8192, 0.98, "magnitude", 32),
        # the largest product of the sweep
        _case("half_8192", 8192, 8192, 0.50, "magnitude", 128),
        # load-balance stress: 16384 x 16384 with Zipf row lengths
        _case("stress", 16384, 16384, 0.95, "zipf", 128),
        # nothing is a multiple of anything, no hint, more columns than one tile
        _case("ragged", 3001, 2511, 0.85, "lognormal", 200, hint=False),
        # new weights arrive (a layer is loaded, a pruning step ends): plan creation and first product
        _case("new_weights", 4096, 4096, 0.80, "magnitude", 64, new_plan=True),
    ]


LARGEST_FLOPS = 2 * 0.5 * 8192 * 8192 * 128
LARGEST_NNZ = 0.5 * 8192 * 8192
LARGEST_BYTES = 8 * LARGEST_NNZ + 8 * 8192 * 128


def draw(rng):
    """Sizes over their logarithm (256 to 16384 rows and columns, 4 to 256 columns of B, densities from
    1/2 to 1/50), one in three a round size, no larger than the largest listed case."""
    def size(lo, hi):
        x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        step = rng.choice((1, 1, 1, 1, 64, 128)) if lo >= 64 else rng.choice((1, 1, 4))
        return int(min(hi, max(lo, round(x / step) * step)))

    while True:
        case = _case("", size(256, 16384), size(256, 16384),
                     round(1.0 - math.exp(rng.uniform(math.log(0.02), math.log(0.5))), 3),
                     rng.choice(("magnitude", "magnitude", "lognormal", "zipf")), size(4, 256),
                     hint=rng.random() < 0.75, keep_out=rng.random() < 0.5, new_plan=rng.random() < 0.1)
        del case["name"]
        w = work(case)
        if w["flops"] <= LARGEST_FLOPS and w["bytes"] <= LARGEST_BYTES:
            return case


def _row_densities(case, seed):
    """Density of every row, as in workloads/generators.py (lognormal_rows, zipf_rows)."""
    M, K, d = case["rows"], case["cols"], 1.0 - case["sparsity"]
    rng = np.random.default_rng(seed)
    if case["law"] == "lognormal":
        return np.clip(d * np.exp(0.5 * rng.standard_normal(M) - 0.125), 0.0, 1.0)
    order = rng.permutation(M)
    live = order[int(round(0.05 * M)):]
    z = np.minimum(rng.zipf(1.5, size=live.size), K).astype(np.float64)
    scale = d * M * K / z.sum()
    for _ in range(8):
        lens = np.clip(scale * z, 1, K)
        if abs(lens.sum() - d * M * K) <= 0.01 * d * M * K:
            break
        scale *= d * M * K / lens.sum()
    dens = np.zeros(M)
    dens[live] = lens / K
    return dens


def _weights(case, seed):
    """A as host CSR arrays (int32 row_ptr and ascending col_idx, float32 vals), drawn on the GPU."""
    M, K = case["rows"], case["cols"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["law"] == "magnitude":
        W = torch.randn((M, K), device="cuda", generator=g)
        cut = float(torch.special.ndtri(torch.tensor(1.0 - 0.5 * (1.0 - case["sparsity"]), dtype=torch.float64)))
        mask = W.abs() > cut
    else:
        dens = torch.from_numpy(_row_densities(case, seed).astype(np.float32)).cuda()
        mask = torch.rand((M, K), device="cuda", generator=g) < dens[:, None]
        W = torch.randn((M, K), device="cuda", generator=g).mul_(0.02 if case["law"] == "lognormal" else 1.0)
    row_ptr = torch.zeros(M + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(mask.sum(dim=1), 0, out=row_ptr[1:])
    col_idx = mask.nonzero()[:, 1].to(torch.int32)
    vals = W[mask]
    return row_ptr.to(torch.int32).cpu().numpy(), col_idx.cpu().numpy(), vals.cpu().numpy()


def _plan(state):
    case = state["case"]
    return spmm.plan_create(case["rows"], case["cols"], *state["csr"], n_hint=case["width"] if case["hint"] else 0)


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed + 1_000_003)
    state = dict(case=case, csr=_weights(case, seed), plan=None, C=None,
                 B=torch.randn((case["cols"], case["width"]), device="cuda", generator=g))
    if case["keep_out"]:
        state["C"] = torch.empty((case["rows"], case["width"]), device="cuda")
    if not case["new_plan"]:
        state["plan"] = _plan(state)
        state["csr"] = None
    return state


def run(state):
    plan = state["plan"] if state["plan"] is not None else _plan(state)
    return plan.execute(state["B"], state["C"])


def work(case):
    M, K, N = case["rows"], case["cols"], case["width"]
    nnz = (1.0 - case["sparsity"]) * M * K
    return {"bytes": 4 * (M + 1) + 8 * nnz + 4 * K * N + 4 * M * N, "flops": 2 * nnz * N}


def tolerance(case):
    # sums of up to some thousand fp32 products in any order
    return {"rel": 2e-6, "max": 4e-5}
