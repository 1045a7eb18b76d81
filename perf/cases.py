"""Timed cases: what a program that uses this library has it do, through the public entry points.

A pass of most cases is one round of the method for W workers in one GPU's memory (store and average the
models, k local steps, line 6), called the way bench.py, the smoke check and the header's comments call it;
the others are Local SGD's blocking average, the scalar diagnostics, and rounds of perceptron workers whose
gradient is a real mini-batch gradient.  Sizes come from synth_inputs.CONFIGS or are generic.

A case is a dict of plain values:
  kind      "round" (built-in quadratic gradient), "external" (the caller's gradient), "local_sgd",
            "diagnostics", "mlp"
  W, d, k   workers, parameters per worker, local steps of one pass
  tensors   0: one flat vector; n: a list of n tensors (log-uniform sizes, packed), bucket_mib the averaging bucket
  aligned   worker rows start on 4 KiB boundaries (as bench.py lays them out); else the stride of plan_layout
  schedule  "overlap", "serial", "fused", "head";  call: "tail" (line 6 inside the last step), "separate", "graph"
"""
import math

import torch

import paper_1906_12043_amd as P

SCHEDULES = {"overlap": P.SCHED_OVERLAP, "serial": P.SCHED_SERIAL, "fused": P.SCHED_FUSED, "head": P.SCHED_HEAD}
SGD = {"lr": 0.05, "momentum": 0.9, "weight_decay": 5e-4, "noise_sigma": 0.01}
CHUNK = 1024


def _case(name, kind, W, d, k, tensors=0, bucket_mib=0, aligned=True, schedule="overlap", call="tail", weighted=False,
          momentum=0.9, bf16=False):
    return dict(name=name, kind=kind, W=W, d=d, k=k, tensors=tensors, bucket_mib=bucket_mib, aligned=aligned, schedule=schedule,
                call=call, weighted=weighted, momentum=momentum, bf16=bf16)


def _mlp(name, W, n_in, n_hidden, n_out, batch, k, call="tail", schedule="overlap"):
    return dict(name=name, kind="mlp", W=W, n_in=n_in, n_hidden=n_hidden, n_out=n_out, batch=batch, k=k, call=call, schedule=schedule)


def listed():
    return [
        # the tiny configuration: four 65 536-parameter workers, plain SGD, a round of a few microseconds of work
        _case("tiny_round", "round", 4, 65536, 4, momentum=0.0),
        # the headline configuration: ResNet18-sized vector, 16 workers
        _case("resnet18_round", "round", 16, 11_200_000, 2),
        # unequal workers (weighted mean, a noise scale per worker) on a ragged vector, the plain five-call round
        _case("weighted_separate", "round", 12, 2_999_999, 4, aligned=False, call="separate", weighted=True),
        # ImageNet-VGG16-sized vector: the largest configuration, a mean larger than the last-level cache
        _case("vgg16_round", "round", 16, 138_000_000, 2),
        # a list of 62 tensors in 25 MiB buckets, 64 workers
        _case("bucketed_round", "round", 64, 11_200_000, 2, tensors=62, bucket_mib=25),
        # synchronous use: one local step per round, mean and line 6 folded into it
        _case("one_step_round", "round", 16, 11_200_000, 1, schedule="head"),
        # gradients of a mixed-precision backward pass, 16-bit
        _case("external_bf16", "external", 16, 11_200_000, 2, bf16=True),
        # Local SGD: k steps, then the blocking average, on a medium list and an odd number of workers
        _case("local_sgd", "local_sgd", 21, 4_000_037, 2, tensors=40, aligned=False),
        # monitoring of a run with many workers: consensus distance, objective and gradient norm
        _case("diagnostics", "diagnostics", 64, 2_800_003, 0),
        # perceptron workers, the benchmark's shape
        _mlp("mlp_round", 16, 3072, 1024, 10, 128, 2),
        # fewer, wider networks with a larger mini-batch, one step per round
        _mlp("mlp_wide", 6, 1024, 2048, 10, 512, 1, call="separate"),
        # small networks, the round replayed from a graph
        _mlp("mlp_small", 4, 768, 192, 10, 128, 2, call="graph"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["round", "round", "round", "external", "local_sgd", "diagnostics", "mlp", "mlp", "mlp"])
    if kind == "mlp":
        while True:
            W, batch = _log_int(rng, 1, 16), 128 * _log_int(rng, 1, 8)
            n_in, n_hidden, n_out = 128 * _log_int(rng, 1, 24), 64 * _log_int(rng, 1, 32), rng.randint(2, 16)
            if n_hidden * (n_out | 1) <= 32768 and W * n_in * n_hidden * max(batch, 128) <= 16 * 3072 * 1024 * 256:
                c = _mlp("", W, n_in, n_hidden, n_out, batch, rng.randint(1, 4), rng.choice(["tail", "separate", "graph"]),
                         rng.choice(["overlap", "overlap", "serial"]))
                break
    else:
        W = _log_int(rng, 1, 64)
        d = _log_int(rng, 4001, min(138_000_000, 900_000_000 // W)) + rng.randint(0, 5)
        tensors = rng.choice([0, 0, rng.randint(2, 62)]) if d > 40_000 else 0
        c = _case("", kind, W, d, rng.randint(1, 4), tensors=tensors, bucket_mib=25 if tensors and rng.random() < 0.5 else 0,
                  aligned=rng.random() < 0.6, schedule=rng.choice(["overlap", "overlap", "serial", "fused", "head"]),
                  call=rng.choice(["tail", "tail", "separate", "graph"]), weighted=rng.random() < 0.3,
                  momentum=rng.choice([0.9, 0.9, 0.9, 0.0]), bf16=rng.random() < 0.5)
    del c["name"]
    return c


# ---- inputs --------------------------------------------------------------------------------------------

def _generator(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000 + salt)
    return g


def _tensor_sizes(case):
    """Log-uniform tensor sizes that sum to d (the list belongs to the case, not to the seed)."""
    n, d = case["tensors"], case["d"]
    if not n:
        return None
    g = torch.Generator()
    g.manual_seed(n * 7919 + d % 100_003)
    raw = torch.exp(torch.rand(n, generator=g, dtype=torch.float64) * math.log(2_400_000 / 64))
    sizes = [max(1, int(v)) for v in raw * ((d - n) / raw.sum())]
    sizes[max(range(n), key=lambda i: sizes[i])] += d - sum(sizes)
    return sizes


def _layout(case):
    """(sizes, stride, [(first memory element, first global index, n)] per tensor)."""
    sizes = _tensor_sizes(case)
    padded, offsets, _ = P.plan_layout(case["d"], sizes, case["bucket_mib"] << 20)
    stride = -(-padded // CHUNK) * CHUNK if case["aligned"] else padded
    runs, at = [], 0
    for off, n in zip(offsets, sizes or [case["d"]]):
        runs.append((off, at, n))
        at += n
    return sizes, stride, runs


def _clear_pads(buf, runs):
    end = 0
    for off, _, n in runs:
        buf[:, end:off] = 0
        end = off + n
    buf[:, end:] = 0
    return buf


def _hyper(case):
    return dict(SGD, momentum=case["momentum"], weight_decay=SGD["weight_decay"] if case["momentum"] else 0.0)


def _worker_weights(case):
    """p_i and the noise scale of workers whose mini-batches differ in size."""
    if not case["weighted"]:
        return None, None
    m = [16 * (1 + (5 * i) % 8) for i in range(case["W"])]
    return ([float(torch.tensor(v / sum(m), dtype=torch.float32)) for v in m],
            [float(torch.tensor(0.05 / math.sqrt(v), dtype=torch.float32)) for v in m])


def _quadratic_inputs(case, seed):
    """Models in mid-training (workers near one another), a live momentum, curvatures and centres."""
    sizes, stride, runs = _layout(case)
    W, dev = case["W"], "cuda"
    x = torch.randn(W, stride, device=dev, generator=_generator(seed, 1)).mul_(0.05)
    x.add_(torch.randn(stride, device=dev, generator=_generator(seed, 2)).mul_(0.5))
    t = {"x": _clear_pads(x, runs)}
    if case["momentum"]:
        t["v"] = _clear_pads(torch.randn(W, stride, device=dev, generator=_generator(seed, 3)).mul_(0.1), runs)
    if case["kind"] == "external":
        g = torch.randn(W, stride, device=dev, generator=_generator(seed, 4)).mul_(0.1)
        t["g"] = g.to(torch.bfloat16) if case["bf16"] else g
    else:
        t["h"] = _clear_pads(torch.rand(W, stride, device=dev, generator=_generator(seed, 5)).mul_(1.5).add_(0.5), runs)
        t["c"] = _clear_pads(torch.randn(W, stride, device=dev, generator=_generator(seed, 6)), runs)
    return sizes, stride, runs, t


def _mlp_theta(case, seed):
    n_in, n_h, n_out = case["n_in"], case["n_hidden"], case["n_out"]
    g = _generator(seed, 7)
    w1 = torch.randn(n_in * n_h, device="cuda", generator=g) * math.sqrt(2.0 / n_in)
    b1 = torch.randn(n_h, device="cuda", generator=g) * 0.05
    w2 = torch.randn(n_h * n_out, device="cuda", generator=g) * math.sqrt(2.0 / n_h)
    return torch.cat([w1, b1, w2, torch.zeros(n_out, device="cuda")])


MLP_SGD = {"lr": 0.01, "momentum": 0.9, "weight_decay": 1e-3}


def prepare(case, seed):
    W = case["W"]
    s_compute, s_avg = torch.cuda.Stream(), torch.cuda.Stream()
    if case["kind"] == "mlp":
        theta = _mlp_theta(case, seed)
        d = theta.numel()
        stride, _, _ = P.plan_layout(d)
        xA = torch.zeros(W, stride, device="cuda")
        xA[:, :d] = theta
        xB, v = torch.zeros_like(xA), torch.zeros_like(xA)
        mean = torch.zeros(stride, device="cuda")
        torch.cuda.synchronize()
        ctx = P.Context(W=W, d=d, stride=stride, xA=xA, xB=xB, v=v, mean=mean, grad=P.GRAD_MLP,
                        mlp=(case["n_in"], case["n_hidden"], case["n_out"], case["batch"]), seed=seed, compute_stream=s_compute,
                        avg_stream=s_avg, **MLP_SGD)
        g = h = c = None
    else:
        sizes, stride, runs, t = _quadratic_inputs(case, seed)
        xA, v, g, h, c = t["x"], t.get("v"), t.get("g"), t.get("h"), t.get("c")
        xB, mean = torch.zeros_like(xA), torch.zeros(stride, device="cuda")
        weights, sigma_w = _worker_weights(case)
        torch.cuda.synchronize()
        ctx = P.Context(W=W, d=case["d"], stride=stride, xA=xA, xB=xB, v=v, mean=mean, h=h, c=c, seed=seed, tensor_numel=sizes,
                        bucket_bytes=case["bucket_mib"] << 20, weights=weights, noise_sigma_w=sigma_w, compute_stream=s_compute,
                        avg_stream=s_avg, grad=P.GRAD_EXTERNAL if case["kind"] == "external" else P.GRAD_QUADRATIC, **_hyper(case))
    ctx.set_schedule(SCHEDULES[case["schedule"]])
    return {"ctx": ctx, "case": dict(case), "xA": xA, "xB": xB, "v": v, "mean": mean, "g": g, "h": h, "c": c,
            "streams": (s_compute, s_avg), "scalar": torch.zeros(1, dtype=torch.float64, device="cuda")}


def run(state):
    ctx, case = state["ctx"], state["case"]
    kind, k = case["kind"], case["k"]
    if kind == "diagnostics":
        distance = ctx.consensus_distance()
        objective, grad_norm_sq = ctx.quadratic_objective()
        return {"distance": distance, "objective": objective, "grad_norm_sq": grad_norm_sq}
    if kind == "local_sgd":
        ctx.local_steps(k)
        ctx.average_apply_fused()
    elif kind == "external":
        step = ctx.external_step_bf16 if case["bf16"] else ctx.external_step
        ctx.average_begin()
        for s in range(k):
            step(state["g"], close_round=(s == k - 1 and case["call"] != "separate"))
        if case["call"] == "separate":
            ctx.average_end_apply()
    elif case["call"] == "graph":
        ctx.graph_round(k, True)
    elif case["call"] == "separate":
        ctx.round(k)
    else:
        ctx.round_fused_tail(k)
    live = state["xA"] if ctx.live_model() == state["xA"].data_ptr() else state["xB"]
    out = {"x": live, "mean": state["mean"]}
    if state["v"] is not None:
        out["v"] = state["v"]
    return out


# ---- the same in 64 bits, plain torch ------------------------------------------------------------------

def _f32(v):
    return float(torch.tensor(v, dtype=torch.float32))


M32 = 0xFFFFFFFF


def _philox(c0, step, worker, tag, seed):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors; counter (index, step, worker, tag), key = seed."""
    c = [c0, torch.full_like(c0, step), torch.full_like(c0, worker), torch.full_like(c0, tag)]
    k0, k1 = seed & M32, (seed >> 32) & M32
    for _ in range(10):
        a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((b >> 32) & M32) ^ c[1] ^ k0, b & M32, ((a >> 32) & M32) ^ c[3] ^ k1, a & M32]
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c


def _normals(n, step, worker, tag, seed):
    """n normals of one stream from index 0: Box-Muller on the word pairs (0,1) and (2,3)."""
    w = _philox(torch.arange(-(-n // 4), device="cuda", dtype=torch.int64), step, worker, tag, seed)
    z = torch.empty(w[0].numel(), 4, device="cuda", dtype=torch.float64)
    for p in (0, 2):
        r = torch.sqrt(-2.0 * torch.log(((w[p] >> 8) + 1).double() * 2.0**-24))
        a = (w[p + 1] >> 8).double() * (2.0**-24 * 2.0 * math.pi)
        z[:, p], z[:, p + 1] = r * torch.cos(a), r * torch.sin(a)
    return z.view(-1)[:n]


def _exact_quadratic(case, seed):
    sizes, stride, runs, t = _quadratic_inputs(case, seed)
    W, d, k, hy = case["W"], case["d"], case["k"], {n: _f32(v) for n, v in _hyper(case).items()}
    weights, sigma_w = _worker_weights(case)
    p = weights or [1.0 / W] * W
    x = t["x"].double()

    def mean_of(x):
        m = torch.zeros(stride, device="cuda", dtype=torch.float64)
        for i in range(W):
            m += p[i] * x[i]
        return m
    if case["kind"] == "diagnostics":
        m = mean_of(x)
        grad = torch.zeros_like(m)
        distance = objective = 0.0
        for i in range(W):
            distance += p[i] * float(((m - x[i]) ** 2).sum())
            e = m - t["c"][i].double()
            he = t["h"][i].double() * e
            objective += 0.5 * p[i] * float((he * e).sum())
            grad += p[i] * he
        return {"distance": distance, "objective": objective, "grad_norm_sq": float((grad ** 2).sum())}
    m = mean_of(x)
    v = t["v"].double() if "v" in t else None
    for i in range(W):
        xi, vi, start = x[i], None if v is None else v[i], x[i].clone()
        for step in range(k):
            if case["kind"] == "external":
                g = _clear_pads(t["g"][i:i + 1].double(), runs)[0]
            else:
                g = t["h"][i].double() * (xi - t["c"][i].double())
                z = _normals(d, step, i, 0, seed)
                s = sigma_w[i] if sigma_w else hy["noise_sigma"]
                for off, at, n in runs:
                    g[off:off + n] += s * z[at:at + n]
            g += hy["weight_decay"] * xi
            if vi is not None:
                vi.mul_(hy["momentum"]).add_(g)
                g = vi
            xi -= hy["lr"] * g
        if case["kind"] != "local_sgd":
            xi += m - start
    if case["kind"] == "local_sgd":
        m = mean_of(x)
        x[:] = m
    return {"x": x, "mean": m} if v is None else {"x": x, "mean": m, "v": v}


def _exact_mlp(case, seed):
    W, n_in, n_h, n_out, B, k = (case[n] for n in ("W", "n_in", "n_hidden", "n_out", "batch", "k"))
    theta = _mlp_theta(case, seed).double()
    d = theta.numel()
    stride, _, _ = P.plan_layout(d)
    lr, mu, wd = (_f32(MLP_SGD[n]) for n in ("lr", "momentum", "weight_decay"))
    x, v = (torch.zeros(W, stride, device="cuda", dtype=torch.float64) for _ in range(2))
    x[:, :d] = theta
    a, b, c = n_in * n_h, n_in * n_h + n_h, n_in * n_h + n_h + n_h * n_out
    m = x.mean(0)
    for i in range(W):
        xi, vi, start = x[i, :d], v[i, :d], x[i, :d].clone()
        for step in range(k):
            X = _normals(B * n_in, step, i, 4, seed).float().double().view(B, n_in)
            words = torch.stack(_philox(torch.arange(B // 4, device="cuda", dtype=torch.int64), step, i, 5, seed), 1).view(-1)
            y = (words * n_out) >> 32
            W1, b1, W2, b2 = xi[:a].view(n_in, n_h), xi[a:b], xi[b:c].view(n_h, n_out), xi[c:]
            A = X @ W1 + b1
            H = A.clamp(min=0)
            dZ = torch.softmax(H @ W2 + b2, 1)
            dZ[torch.arange(B, device="cuda"), y] -= 1.0
            dZ /= B
            dA = (dZ @ W2.T.contiguous()) * (A > 0)
            g = torch.cat([(X.T.contiguous() @ dA).view(-1), dA.sum(0), (H.T.contiguous() @ dZ).view(-1), dZ.sum(0)]) + wd * xi
            vi.mul_(mu).add_(g)
            xi -= lr * vi
        xi += m[:d] - start
    return {"x": x, "mean": m, "v": v}


def exact(case, seed):
    if case["kind"] != "mlp":
        return _exact_quadratic(case, seed)
    # A unit whose pre-activation lies within rounding of zero may be on or off in a correct 32-bit evaluation, and
    # one such unit outweighs every rounding error in the updated state: where more than a few in a hundred runs
    # meet one, the state in 64 bits says nothing about precision.
    units = case["k"] * case["W"] * case["batch"] * case["n_hidden"]
    out = _exact_mlp(case, seed)
    return out if units * math.sqrt(case["n_in"]) * 4e-9 < 0.03 else {"x": None, "mean": out["mean"], "v": None}


def work(case):
    W, k = case["W"], case["k"]
    if case["kind"] == "mlp":
        n_in, n_h, n_out, B = (case[n] for n in ("n_in", "n_hidden", "n_out", "batch"))
        d = n_in * n_h + n_h + n_h * n_out + n_out
        return {"bytes": (16.0 * W + 4) * d, "flops": k * W * B * (4.0 * n_in * n_h + 6.0 * n_h * n_out)}
    n = float(W) * case["d"]
    if case["kind"] == "diagnostics":                       # read x, h, c
        return {"bytes": 12 * n, "flops": 15 * n}
    state = 16 if case["momentum"] else 8                   # x and v in and out
    grad = (2 if case["bf16"] else 4) if case["kind"] == "external" else 8
    return {"bytes": (state + grad) * n + 4 * case["d"], "flops": (k * (10 if case["kind"] == "external" else 100) + 6) * n}


def tolerance(case):
    if case["kind"] == "mlp":
        # relu decisions within rounding of zero (see exact): one unit taken the other way changes one column
        return {"rel": 1e-2, "max": 1.0}
    if case["kind"] == "diagnostics":
        return {"rel": 1e-6}
    return {"rel": 4e-7}
