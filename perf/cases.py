"""The work that a user of this library has it do, as cases that can be timed.

``listed()`` names them, ``draw(rng)`` gives one more of the same ranges,
``prepare`` makes what a program holds before the call, ``run`` is one pass
through the public entry points, ``work`` the bytes and operations it cannot do
without and ``exact`` its outputs in 64 bits.

Five forms:
* ``mttkrp``   -- one MTTKRP along every mode of a resident tensor, each into its
                  own output, all from the same factors (fp32 or bfloat16 factors);
* ``stream``   -- the same with the layouts in host memory, copied in shards;
* ``oneshot``  -- a tensor built from a COO in host memory, used for one MTTKRP
                  along every mode and closed;
* ``train``    -- the differentiable CP loss: forward and the gradients of all factors;
* ``als``      -- a CP-ALS sweep from a program's initial factors, which it keeps.

Tensors have distinct coordinates, sorted as files have them, with Zipf or uniform
indices per mode (Zipf ranks are scattered over the index space), values in (0, 1)
and factors in (-1, 1), the inputs that the benchmark and the tests use.
"""
import math

import numpy as np
import torch

from paper_2507_15121_amd import api
from paper_2507_15121_amd.autograd import sparse_cp_loss

DEVICE = "cuda"


def _case(name, form, dims, nnz, rank, dtype="f32", s=0.0, hot=0.0, sorted_input=True, shard=0):
    return {"name": name, "form": form, "dims": "x".join(str(d) for d in dims), "nnz": nnz, "rank": rank,
            "dtype": dtype, "zipf": s, "hot": hot, "sorted": sorted_input, "shard": shard}


def listed():
    return [
        # the smallest calls: a tensor of a few hundred rows, where a call is its launches and one pass's latency
        _case("mttkrp-tiny-o4-r16", "mttkrp", (30, 20, 10, 8), 2000, 16),
        # the benchmark's small workload, a tensor that fits every cache
        _case("mttkrp-100k-r16", "mttkrp", (1000, 800, 600), 100_000, 16),
        # an ordinary tensor: factors beyond the L2, a hundred nonzeros for each SIMD lane
        _case("mttkrp-5M-r32", "mttkrp", (250_000, 125_000, 50_000), 5_000_000, 32, s=1.1),
        # ranks are chosen by the model, not by the vector width; ragged mode sizes
        _case("mttkrp-3M-r20", "mttkrp", (100_003, 70_001, 3_001), 3_000_000, 20, s=1.1),
        # bfloat16 factors, rank 64 (rows of 128 bytes), one heavy slice
        _case("mttkrp-20M-r64-bf16", "mttkrp", (1_000_000, 500_000, 200_000), 20_000_000, 64, "bf16", s=1.1, hot=0.05),
        # the benchmark's 200M-nonzero workload, the largest here
        _case("mttkrp-200M-r32", "mttkrp", (10_000_000, 5_000_000, 2_000_000), 200_000_000, 32, s=1.1),
        # layouts kept in host memory, for tensors beyond the device's: the host link is the path
        _case("stream-10M-r32", "stream", (500_000, 250_000, 100_000), 10_000_000, 32, s=1.1, shard=1 << 21),
        # a program that decomposes many tensors once each: the build is part of every answer
        _case("oneshot-5M-r32", "oneshot", (250_000, 125_000, 50_000), 5_000_000, 32, s=1.1, sorted_input=False),
        # gradient training on a small and on a large order-4 tensor
        _case("train-100k-r16", "train", (1000, 800, 600), 100_000, 16),
        _case("train-10M-o4-r32", "train", (1_000_000, 400_000, 20_000, 2_000), 10_000_000, 32, s=1.2),
        # alternating least squares on a small and on a large tensor
        _case("als-100k-r16", "als", (1000, 800, 600), 100_000, 16),
        _case("als-10M-r32", "als", (500_000, 250_000, 100_000), 10_000_000, 32, s=1.1),
    ]


# the ranks of the tests and the benchmark, and others that models use
RANKS = (5, 8, 10, 16, 20, 24, 25, 32, 32, 48, 50, 64, 100, 128)


def draw(rng):
    form = rng.choice(("mttkrp", "mttkrp", "mttkrp", "mttkrp", "stream", "oneshot", "train", "train", "als", "als"))
    order = rng.choice((2, 3, 3, 3, 4, 4, 5))
    rank = rng.choice(RANKS)
    if form == "train":
        rank = rng.choice([r for r in RANKS if r <= 64])
    # nonzeros: every form's pass stays below the largest listed one's cost
    low, high = (2_000, 20_000_000) if form == "mttkrp" else (100_000, 5_000_000)
    high = min(high, int(high * 32 / rank))
    nnz = int(math.exp(rng.uniform(math.log(low), math.log(high))))
    # mode sizes: the first modes a few percent of the nonzeros, as large as the factors' rows allow, the later
    # ones smaller, all of them odd as often as not
    dims = []
    for w in range(order):
        share = math.exp(rng.uniform(math.log(0.002), math.log(0.3))) * 0.5 ** w
        least = 2 * rank if form == "als" else 8   # least squares for more unknowns than rows has no single answer
        dims.append(max(least + rng.randrange(8), int(nnz * share) + rng.randrange(2)))
    # the index space holds at least eight times the nonzeros (distinct coordinates)
    while math.prod(dims) < 8 * nnz:
        dims[0] = 2 * dims[0] + 1
    zipf = rng.choice((0.0, 1.1, 1.1, 1.2))
    if math.prod(dims) < 4000 * nnz:
        zipf = 0.0   # too dense for distinct coordinates of a power law
    case = _case("", form, dims, nnz, rank, "bf16" if form == "mttkrp" and rng.random() < 0.35 else "f32", zipf,
                 0.05 if zipf and rng.random() < 0.3 else 0.0, rng.random() < 0.5,
                 1 << rng.randrange(17, 21) if form == "stream" else 0)
    del case["name"]
    return case


def _dims(case):
    return [int(d) for d in case["dims"].split("x")]


# ------------------------------------------------------------------ inputs

def _cdf(rows, s):
    c = np.cumsum(np.arange(1, rows + 1, dtype=np.float64) ** -s)   # on the host: the same bits every time
    return torch.from_numpy(c / c[-1]).to(DEVICE)


def _draws(case, gen, n, tables):
    """n index tuples, [order] int32 tensors."""
    out = []
    for d, table in zip(_dims(case), tables):
        if table is None:
            out.append(torch.randint(d, (n,), generator=gen, device=DEVICE, dtype=torch.int32))
        else:
            cdf, scatter = table
            u = torch.rand(n, generator=gen, device=DEVICE, dtype=torch.float64)
            out.append(scatter[torch.searchsorted(cdf, u).clamp_(max=d - 1)])
    if case["hot"]:
        out[0][torch.rand(n, generator=gen, device=DEVICE) < case["hot"]] = _dims(case)[0] // 2
    return out


def _coo(case, gen):
    """Distinct coordinates (the first nnz in draw order) in lexicographic
    order, int32 [order, nnz], and their values, on the GPU."""
    dims, nnz = _dims(case), case["nnz"]
    tables = [None] * len(dims)
    if case["zipf"]:
        tables = [(_cdf(d, case["zipf"]), torch.randperm(d, generator=gen, device=DEVICE).to(torch.int32)) for d in dims]
    cols = None
    n = int(nnz * (1.6 if case["zipf"] else 1.15)) + 64
    while True:
        more = _draws(case, gen, n, tables)
        cols = more if cols is None else [torch.cat(p) for p in zip(cols, more)]
        total = cols[0].numel()
        # stable sorts, the last modes first, as many modes to a key as fit in 62 bits
        order = None
        first = torch.zeros(total, dtype=torch.bool, device=DEVICE)
        first[:1] = True
        w = len(dims)
        while w > 0:
            key, bits = None, 0
            at = w
            while at > 0 and bits + (dims[at - 1] - 1).bit_length() <= 62:
                at -= 1
                part = cols[at].long() << bits
                key = part if key is None else key.add_(part)
                bits += (dims[at] - 1).bit_length()
            if order is None:
                order = torch.sort(key, stable=True)[1]
            else:
                order = order[torch.sort(key[order], stable=True)[1]]
            w = at
            del key
        for c in cols:
            c = c[order]
            first[1:] |= c[1:] != c[:-1]
        ids = order[first]
        del order, first
        if ids.numel() >= nnz:
            break
    fresh = torch.zeros(total, dtype=torch.bool, device=DEVICE)
    fresh[ids] = True
    fresh &= torch.cumsum(fresh, 0) <= nnz
    ids = ids[fresh[ids]]
    del fresh
    if not case["sorted"]:
        ids = ids[torch.randperm(nnz, generator=gen, device=DEVICE)]
    idx = torch.stack([c[ids] for c in cols])
    return idx, torch.rand(nnz, generator=gen, device=DEVICE).clamp_(min=1e-6)


def _factors(case, gen):
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    return [(torch.rand((d, case["rank"]), generator=gen, device=DEVICE) * 2 - 1).to(dtype) for d in _dims(case)]


def _inputs(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    idx, val = _coo(case, gen)
    return idx, val, _factors(case, gen)


def prepare(case, seed):
    dims, form, rank = _dims(case), case["form"], case["rank"]
    idx, val, factors = _inputs(case, seed)
    idx, val = idx.cpu().numpy(), val.cpu().numpy()
    torch.cuda.empty_cache()
    state = {"form": form, "dims": dims, "factors": factors, "bf16": case["dtype"] == "bf16"}
    if form == "oneshot":
        state["coo"] = (idx, val)
    elif form == "stream":
        state["tensor"] = api.Tensor(idx, val, dims, host_layout=True, shard_nnz=case["shard"])
    else:
        state["tensor"] = api.Tensor(idx, val, dims)
    if form == "train":
        for f in factors:
            f.requires_grad_(True)
    elif form == "als":
        state["current"] = [torch.empty_like(f) for f in factors]
        state["weights"] = torch.empty(rank, dtype=torch.float64, device=DEVICE)
        state["fit"] = torch.empty((), dtype=torch.float64, device=DEVICE)
    else:
        state["outs"] = [torch.empty((d, rank), device=DEVICE) for d in dims]
    return state


# -------------------------------------------------------------------- one pass

def _all_modes(tensor, state):
    call = api.mttkrp_bf16 if state["bf16"] else api.mttkrp
    for d, out in enumerate(state["outs"]):
        call(tensor, d, state["factors"], out=out)
    return state["outs"]


def run(state):
    form = state["form"]
    if form == "oneshot":
        tensor = api.Tensor(*state["coo"], state["dims"])
        outs = _all_modes(tensor, state)
        tensor.close()
        return outs
    if form == "train":
        factors = state["factors"]
        for f in factors:
            f.grad = None
        loss = sparse_cp_loss(state["tensor"], *factors)
        loss.backward()
        return {"loss": loss.detach(), "grads": [f.grad for f in factors]}
    if form == "als":
        current = state["current"]
        for c, f in zip(current, state["factors"]):
            c.copy_(f)
        api.cp_als_sweep(state["tensor"], current, state["weights"], state["fit"])
        # the model as a program keeps it, in its factors' type
        return {"factors": current, "weights": state["weights"].float(), "fit": state["fit"].float()}
    return _all_modes(state["tensor"], state)


# ------------------------------------------------------------------------ work

def _distinct(rows, nnz, s):
    """Expected distinct indices of a mode."""
    if not s:
        return rows * -math.expm1(-nnz / rows)
    k = np.arange(1, rows + 1, dtype=np.float64) ** -s
    return float(-np.expm1(k * (-nnz / k.sum())).sum())


def work(case):
    """Each call's inputs read once and its outputs written once: the nonzeros
    (indices and value), the distinct factor rows that they name, the output."""
    dims, nnz, r, n = _dims(case), case["nnz"], case["rank"], len(_dims(case))
    size = 2 if case["dtype"] == "bf16" else 4
    used = [_distinct(d, nnz, case["zipf"]) * r * size for d in dims]
    tensor = nnz * (4.0 * n + 4)
    if case["form"] == "train":
        # loss and all gradients from the nonzeros and the factor rows
        return {"bytes": tensor + sum(used) + sum(dims) * r * 4.0, "flops": nnz * r * (n + 1.0) * n}
    step_bytes = n * tensor + (n - 1) * sum(used) + sum(dims) * r * 4.0
    step_flops = float(nnz) * r * n * n
    if case["form"] == "als":
        # the copy of the initial factors and their Gram matrices, then each mode's MTTKRP, its output's Gram matrix
        # and the new factor
        rows = sum(dims) * r
        return {"bytes": step_bytes + 12.0 * rows, "flops": step_flops + 6.0 * rows * r}
    return {"bytes": step_bytes, "flops": step_flops}


# ------------------------------------------------------------------ in 64 bits

def _sum_by_row(row, p):
    """Sums of p's rows that share a value of the sorted row[], in runs of at
    most 64 terms at a time: (distinct values, their sums)."""
    while True:
        place = torch.arange(row.numel(), device=DEVICE)
        new = torch.ones_like(place, dtype=torch.bool)
        new[1:] = row[1:] != row[:-1]
        place -= torch.cummax(place * new, 0)[0]   # within its row
        at = torch.nonzero(place % 64 == 0)[:, 0]
        ends = torch.cat([at[1:], torch.full_like(at[:1], row.numel())])
        p = torch.segment_reduce(p, "sum", lengths=ends - at, axis=0)
        row = row[at]
        if not bool((row[1:] == row[:-1]).any()):
            return row, p


def _exact_mttkrp(idx, val, factors, mode, rows):
    rank = factors[0].shape[1]
    out = torch.zeros((rows, rank), dtype=torch.float64, device=DEVICE)
    order = torch.sort(idx[mode], stable=True)[1]
    piece = max(64, (1 << 28) // rank)
    for a in range(0, val.numel(), piece):
        at = order[a:a + piece]
        p = val[at].double()[:, None].expand(-1, rank)
        for w, f in enumerate(factors):
            if w != mode:
                p = p * f[idx[w, at].long()].double()
        row, p = _sum_by_row(idx[mode, at].long(), p)
        out[row] += p
    return out


def _exact_residuals(idx, val, factors):
    rank = factors[0].shape[1]
    e = val.double()
    piece = max(1, (1 << 28) // rank)
    for a in range(0, val.numel(), piece):
        b = a + piece
        p = None
        for w, f in enumerate(factors):
            g = f[idx[w, a:b].long()].double()
            p = g if p is None else p * g
        e[a:b] -= p.sum(1)
    return e


def exact(case, seed):
    idx, val, factors = _inputs(case, seed)
    dims, n = _dims(case), len(_dims(case))
    if case["form"] == "train":
        e = _exact_residuals(idx, val, factors)
        return {"loss": e.square().sum(),
                "grads": [-2.0 * _exact_mttkrp(idx, e, factors, d, dims[d]) for d in range(n)]}
    if case["form"] == "als":
        a = [f.double() for f in factors]
        x2 = val.double().square().sum()
        grams = [f.t() @ f for f in a]
        for d in range(n):
            m = _exact_mttkrp(idx, val, a, d, dims[d])
            v = torch.ones_like(grams[0])
            for w in range(n):
                if w != d:
                    v = v * grams[w]
            new = torch.linalg.solve(v, m.t()).t()
            weights = new.norm(dim=0)
            a[d] = torch.where(weights > 0, new / weights, torch.zeros_like(new))
            grams[d] = a[d].t() @ a[d]
        inner = (m * (a[n - 1] * weights)).sum()
        full = torch.ones_like(grams[0])
        for g in grams:
            full = full * g
        model2 = weights @ full @ weights
        fit = 1.0 - (x2 - 2.0 * inner + model2).clamp(min=0.0).sqrt() / x2.sqrt()
        return {"factors": a, "weights": weights, "fit": fit}
    return [_exact_mttkrp(idx, val, factors, d, dims[d]) for d in range(n)]
