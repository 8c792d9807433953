"""The work that a user of libmhlmoe has it do, as cases to measure.

A case is one shape (T tokens, n_heads, d_head, n_experts, top_k, d_ff, dtype,
expert form, bias) and one path through the public entry points:

  forward          one layer forward (routing and experts)
  train            the layer forward and its backward on the forward's routing
  backward         the layer backward on a routing kept from the forward
  routing          routing alone, forward and backward (Algorithms 1 and 2)
  latent           the layer between its projections, with separate routing
                   sub-tokens, forward
  latent_backward  the backward of that

The inputs follow workloads.py: X, dY ~ N(0, 1); W_router, W1, W3 ~ N(0,
1/d_head); W2 ~ N(0, 1/d_ff); the Zipf bias -s ln(1 + rank) with s = 1.1; they
are drawn on the GPU.  Workspaces and output buffers are allocated once and
kept, as a training or serving loop keeps them.
"""
import math

import torch

import paper_2602_04870_amd as mh

ZIPF_S = 1.1


def _case(path, T, n_heads, d_head, n_experts, top_k, d_ff, dtype="bf16", expert="swiglu",
          bias="none", d_model=0, name=None):
    c = dict(path=path, T=T, n_heads=n_heads, d_head=d_head, n_experts=n_experts, top_k=top_k,
             d_ff=d_ff, dtype=dtype, expert=expert, bias=bias, d_model=d_model)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # fp32 users: the oracle-sized layer, bound by launches and latency
        _case("forward", 256, 4, 64, 16, 2, 128, "f32", name="tiny_f32_forward"),
        # serving: one small batch of decoded tokens through a trained layer,
        # a few slots per expert
        _case("forward", 96, 8, 128, 64, 8, 256, name="decode_t96_forward"),
        # the default benchmark: one 4096-token sequence, 512 slots per expert
        _case("forward", 4096, 8, 128, 64, 8, 256, name="t4096_e64_forward"),
        # the same layer in training: the backward on the kept routing
        _case("backward", 4096, 8, 128, 64, 8, 256, name="t4096_e64_backward"),
        # prefill of the larger model: 16 heads, 128 experts
        _case("forward", 16384, 16, 128, 128, 8, 256, name="headline_forward"),
        # one training step of it
        _case("train", 16384, 16, 128, 128, 8, 256, name="headline_train"),
        # doubled granularity: twice the experts of half the width, k 16
        _case("forward", 16384, 16, 128, 256, 16, 128, name="granular_forward"),
        # the skewed training workload: 1024 experts, k 32, Zipf load
        _case("train", 65536, 8, 128, 1024, 32, 128, bias="zipf", name="skewed_train"),
        # the paper's own expert (two matrices, GELU) at its 384-expert layer,
        # four 2048-token sequences: about 85 slots per expert
        _case("train", 8192, 8, 128, 384, 4, 256, expert="gelu", name="gelu_e384_train"),
        # odd sizes: ragged batch, narrow heads, expert count and d_ff that
        # are no multiple of the tiles
        _case("train", 3001, 5, 64, 100, 5, 96, bias="zipf", name="ragged_d64_train"),
        # the routing sweep of the per-component analysis, at 512 experts
        _case("routing", 40000, 8, 128, 512, 8, 32, name="routing_e512"),
        # the layer with its projections and separate routing sub-tokens
        _case("latent", 4096, 8, 128, 64, 8, 256, d_model=1024, name="latent_t4096_forward"),
    ]


def _largest():
    return _cost(listed()[7])


def _cost(c):
    # work() plus the per-slot rows, which bound the memory a case needs
    w = work(c)
    return max(w["flops"] / 5e14, w["bytes"] / 4e12)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        path = rng.choice(["forward", "forward", "forward", "train", "train", "backward", "routing",
                           "latent", "latent_backward"])
        dtype = "f32" if path in ("forward", "routing") and rng.random() < 0.15 else "bf16"
        n_experts = _log_int(rng, 8, 1024)
        c = _case(path, _log_int(rng, 64, 65536), rng.choice([1, 2, 3, 4, 5, 8, 8, 12, 16]),
                  rng.choice([64, 128, 128]), n_experts,
                  min(n_experts, rng.choice([1, 2, 3, 4, 5, 6, 8, 8, 12, 16, 24, 32])),
                  rng.choice([32, 64, 96, 128, 128, 160, 192, 256, 256, 320, 384, 512]), dtype,
                  rng.choice(["swiglu", "swiglu", "gelu"]), rng.choice(["none", "none", "zipf"]),
                  8 * rng.randint(16, 256) if path.startswith("latent") else 0)
        if path == "routing":
            c["d_ff"] = 32
            c["expert"] = "swiglu"
        if _cost(c) <= 0.5 * _largest():
            return c


def _torch_dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _shape(c):
    return c["T"], c["n_heads"], c["d_head"], c["n_experts"], c["top_k"], c["d_ff"]


def _plain_routing(R, W_router, bias, k):
    """idx and gate of plain torch in fp32, as a forward pass left them."""
    T, Nh, _ = R.shape
    idx = torch.empty((T, Nh, k), dtype=torch.int32, device=R.device)
    gate = torch.empty((T, Nh, k), dtype=torch.float32, device=R.device)
    for h in range(Nh):
        s = R[:, h].float() @ W_router[h].t()
        top = torch.topk(s if bias is None else s + bias[h], k, dim=1).indices
        idx[:, h] = top.to(torch.int32)
        gate[:, h] = torch.softmax(torch.gather(s, 1, top), dim=1)
    return idx, gate


def _inputs(c, seed):
    T, Nh, dh, Ne, k, dff = _shape(c)
    dt = _torch_dtype(c)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(shape, std, dtype):
        return (torch.randn(shape, generator=gen, device="cuda") * std).to(dtype)

    s = {"X": None, "W_router": None, "bias": None, "W1": None, "W3": None, "W2": None}
    if not c["d_model"]:
        s["X"] = normal((T, Nh, dh), 1.0, dt)
    s["W_router"] = normal((Nh, Ne, dh), dh ** -0.5, torch.float32)
    if c["bias"] == "zipf":
        rank = torch.stack([torch.randperm(Ne, generator=gen, device="cuda") for _ in range(Nh)])
        s["bias"] = -ZIPF_S * torch.log1p(rank.float())
    if c["path"] != "routing":
        s["W1"] = normal((Nh, Ne, dff, dh), dh ** -0.5, dt)
        if c["expert"] == "swiglu":
            s["W3"] = normal((Nh, Ne, dff, dh), dh ** -0.5, dt)
        s["W2"] = normal((Nh, Ne, dh, dff), dff ** -0.5, dt)
    if c["path"] in ("train", "backward"):
        s["dY"] = normal((T, Nh, dh), 1.0, dt)
    if c["path"] == "backward":
        s["idx"], s["gate"] = _plain_routing(s["X"], s["W_router"], s["bias"], k)
    if c["path"] == "routing":
        s["dgate"] = normal((T, Nh, k), 1.0, torch.float32)
    if c["d_model"]:
        dm, N = c["d_model"], Nh * dh
        s["x"] = normal((T, dm), 1.0, dt)
        s["W_in"] = normal((2 * N, dm), dm ** -0.5, dt)
        s["W_out"] = normal((dm, N), N ** -0.5, dt)
        if c["path"] == "latent_backward":
            s["dout"] = normal((T, dm), 1.0, dt)
            s["X_lat"], s["R_lat"], s["Y_lat"] = (normal((T, Nh, dh), 1.0, dt) for _ in range(3))
            s["idx"], s["gate"] = _plain_routing(s["R_lat"], s["W_router"], s["bias"], k)
    return s


def prepare(case, seed):
    c = case
    T, Nh, dh, Ne, k, dff = _shape(c)
    dt = _torch_dtype(c)
    s = _inputs(c, seed)
    s["case"] = c
    code = mh.MHLMOE_F32 if c["dtype"] == "f32" else mh.MHLMOE_BF16

    def buf(shape, dtype):
        return torch.empty(shape, dtype=dtype, device="cuda")

    f32 = torch.float32
    # the workspaces that a loop over this shape keeps
    names = {"routing": ["ROUTE", "ROUTE_BACKWARD"], "forward": ["LAYER"], "backward": ["LAYER_BACKWARD"],
             "train": ["LAYER", "LAYER_BACKWARD"], "latent": ["LATENT_LAYER"],
             "latent_backward": ["LATENT_BACKWARD"]}[c["path"]]
    n = max(mh.mhlmoe_workspace_size(getattr(mh, "MHLMOE_OP_" + o), T, Nh, dh, Ne, k, dff, code) for o in names)
    s["ws"] = buf((max(n, 256),), torch.uint8)
    if c["path"] in ("forward", "train", "routing", "latent"):
        s["routing"] = dict(idx=buf((T, Nh, k), torch.int32), gate=buf((T, Nh, k), f32),
                            counts=buf((Nh, Ne), torch.int32))
    if c["path"] in ("forward", "train"):
        s["Y"] = buf((T, Nh, dh), dt)
    if c["path"] in ("backward", "train"):
        g = dict(dX=buf((T, Nh, dh), dt), dW_router=buf((Nh, Ne, dh), f32))
        if c["expert"] == "gelu":
            g.update(dW_in=buf((Nh, Ne, dff, dh), f32), dW_out=buf((Nh, Ne, dh, dff), f32))
        else:
            g.update(dW1=buf((Nh, Ne, dff, dh), f32), dW3=buf((Nh, Ne, dff, dh), f32),
                     dW2=buf((Nh, Ne, dh, dff), f32))
        s["grads"] = g
    if c["path"] == "routing":
        s["grads"] = dict(dX=buf((T, Nh, dh), dt), dW_router=buf((Nh, Ne, dh), f32))
    if c["path"] == "latent":
        s["acts"] = dict(out=buf((T, c["d_model"]), dt), X_lat=buf((T, Nh, dh), dt),
                         R_lat=buf((T, Nh, dh), dt), Y_lat=buf((T, Nh, dh), dt))
    return s


def _forward(s):
    c = s["case"]
    if c["expert"] == "gelu":
        return mh.mhlmoe_layer_gelu(s["X"], s["W_router"], s["bias"], s["W1"], s["W2"], c["top_k"],
                                    Y=s["Y"], workspace=s["ws"], **s["routing"])
    return mh.mhlmoe_layer(s["X"], s["W_router"], s["bias"], s["W1"], s["W3"], s["W2"], c["top_k"],
                           Y=s["Y"], workspace=s["ws"], **s["routing"])


def _backward(s, idx, gate):
    if s["case"]["expert"] == "gelu":
        return mh.mhlmoe_layer_gelu_backward(s["X"], s["W_router"], s["W1"], s["W2"], idx, gate,
                                             s["dY"], workspace=s["ws"], **s["grads"])
    return mh.mhlmoe_layer_backward(s["X"], s["W_router"], s["W1"], s["W3"], s["W2"], idx, gate,
                                    s["dY"], workspace=s["ws"], **s["grads"])


def run(state):
    s, path = state, state["case"]["path"]
    if path == "forward":
        return list(_forward(s))
    if path == "backward":
        return list(_backward(s, s["idx"], s["gate"]))
    if path == "train":
        Y, idx, gate, counts = _forward(s)
        return [Y, idx, gate, counts, *_backward(s, idx, gate)]
    if path == "routing":
        idx, gate, counts = mh.mhlmoe_route(s["X"], s["W_router"], s["bias"], s["case"]["top_k"],
                                            workspace=s["ws"], **s["routing"])
        return [idx, gate, counts,
                *mh.mhlmoe_route_backward(s["X"], s["W_router"], idx, gate, s["dgate"],
                                          workspace=s["ws"], **s["grads"])]
    if path == "latent":
        r = mh.mhlmoe_latent_layer(s["x"], s["W_in"], s["W_router"], s["bias"], s["W1"], s["W3"],
                                   s["W2"], s["W_out"], s["case"]["n_heads"], s["case"]["top_k"],
                                   routing_tokens=True, workspace=s["ws"], **s["acts"],
                                   **s["routing"])
        return [r[n] for n in ("out", "X_lat", "R_lat", "Y_lat", "idx", "gate", "counts")]
    g = mh.mhlmoe_latent_layer_backward(s["x"], s["W_in"], s["W_router"], s["W1"], s["W3"], s["W2"],
                                        s["W_out"], s["X_lat"], s["R_lat"], s["Y_lat"], s["idx"],
                                        s["gate"], s["dout"], routing_tokens=True,
                                        workspace=s["ws"])
    return [g[n] for n in ("dx", "dW_in", "dW_router", "dW1", "dW3", "dW2", "dW_out")
            if g[n] is not None]


def work(case):
    """Operands read once, results written once, and the multiply-adds of the
    products (two operations each).  Per slot and d_head x d_ff matrix: the
    forward uses each matrix once; the backward needs the recomputed
    intermediate (W1, W3), W2^T dy, the input gradient (W1, W3) and one outer
    product per matrix."""
    c = case
    T, Nh, dh, Ne, k, dff = _shape(c)
    e = 4 if c["dtype"] == "f32" else 2
    mats = 2 if c["expert"] == "gelu" else 3
    slots = T * Nh * k
    rows = T * Nh * dh * e
    # experts without a slot need neither their weights nor any gradient work
    used = min(Nh * Ne, slots)
    weights = used * mats * dh * dff * e
    router = Nh * Ne * dh * 4
    routing = 8 * slots + 4 * Nh * Ne
    mac = 2 * dh * dff * slots
    fwd_flops = 2 * T * Nh * Ne * dh + mats * mac
    fwd_bytes = 2 * rows + router + weights + routing
    bwd_flops = (2 * (mats - 1) + 1 + mats) * mac + 4 * slots * dh
    bwd_bytes = 3 * rows + 2 * router + weights + 8 * slots + Nh * Ne * mats * dh * dff * 4
    if c["path"] == "forward":
        return {"bytes": fwd_bytes, "flops": fwd_flops}
    if c["path"] == "backward":
        return {"bytes": bwd_bytes, "flops": bwd_flops}
    if c["path"] == "train":
        return {"bytes": fwd_bytes + bwd_bytes, "flops": fwd_flops + bwd_flops}
    if c["path"] == "routing":
        return {"bytes": 3 * rows + 3 * router + 2 * routing + 4 * slots,
                "flops": 2 * T * Nh * Ne * dh + 4 * slots * dh}
    dm, N = c["d_model"], Nh * dh
    act, proj = T * dm * e, 3 * N * dm * e
    if c["path"] == "latent":
        return {"bytes": fwd_bytes + rows + 2 * act + proj, "flops": fwd_flops + 6 * T * N * dm}
    return {"bytes": bwd_bytes + 2 * rows + 3 * act + 3 * proj,
            "flops": bwd_flops + 12 * T * N * dm}


def tolerance(case):
    # Set beside measured figures: against 64 bits the bf16 paths are 2e-3 to
    # 4e-3 off (three roundings to bf16 on the way) and the fp32 ones 2e-7 to
    # 5e-7.  A routing decision between two experts whose scores differ by the
    # router's own rounding may fall either way in another implementation
    # (about 1e-4 of the rows), which moves that row by up to its own size.
    if case["dtype"] == "f32":
        return {"rel": 1e-5 if case["path"] == "forward" else 2e-5, "max": 0.9, "differ": 2e-3}
    if case["path"] == "backward":
        return {"rel": 1e-2, "max": 0.2}
    return {"rel": 1.2e-2, "max": 0.9, "differ": 2e-3}


def _act(c, a):
    """(value, derivative) of the activation in 64 bits."""
    if c["expert"] == "gelu":
        cdf = 0.5 * torch.erfc(-a / math.sqrt(2.0))
        return a * cdf, cdf + a * torch.exp(-0.5 * a * a) / math.sqrt(2.0 * math.pi)
    g = torch.sigmoid(a)
    return a * g, g * (1.0 + a * (1.0 - g))


def _experts64(c, s, X, idx, gate, h, dY=None):
    """One head in 64 bits: Y, and with dY also (dX, dgate, dW1, dW3, dW2)."""
    T, Nh, dh, Ne, k, dff = _shape(c)
    f64 = torch.float64
    Y = torch.zeros((T, dh), dtype=f64, device="cuda")
    order = torch.argsort(idx.reshape(-1), stable=True)
    ends = torch.cumsum(torch.bincount(idx.reshape(-1), minlength=Ne), 0).tolist()
    gf = gate.reshape(-1)
    if dY is not None:
        dX = torch.zeros((T, dh), dtype=f64, device="cuda")
        dgate = torch.zeros(T * k, dtype=f64, device="cuda")
        dW = [torch.zeros((Ne, dff, dh), dtype=f64, device="cuda"),
              torch.zeros((Ne, dff, dh), dtype=f64, device="cuda") if s["W3"] is not None else None,
              torch.zeros((Ne, dh, dff), dtype=f64, device="cuda")]
    for e in range(Ne):
        slots = order[(ends[e - 1] if e else 0):ends[e]]
        if not len(slots):
            continue
        tok = slots // k
        x, g = X[tok], gf[slots][:, None]
        W1, W2 = s["W1"][h, e].to(f64), s["W2"][h, e].to(f64)
        a = x @ W1.t()
        f, df = _act(c, a)
        u = f
        if s["W3"] is not None:
            W3 = s["W3"][h, e].to(f64)
            b = x @ W3.t()
            u = f * b
        if dY is None or c["path"] == "train":
            Y.index_add_(0, tok, g * (u @ W2.t()))
        if dY is not None:
            dy = dY[tok]
            v = dy @ W2
            dgate[slots] = (v * u).sum(1)
            du = g * v
            if s["W3"] is not None:
                da, db = du * b * df, du * f
                dW[1][e] = db.t() @ x
                dx = da @ W1 + db @ W3
            else:
                da = du * df
                dx = da @ W1
            dW[0][e] = da.t() @ x
            dW[2][e] = dy.t() @ (g * u)
            dX.index_add_(0, tok, dx)
    if dY is None:
        return Y
    return Y, dX, dgate.reshape(T, k), dW


def _route64(c, s, R, h):
    """(idx, gate) of one head in 64 bits."""
    sc = R @ s["W_router"][h].to(torch.float64).t()
    key = sc if s["bias"] is None else sc + s["bias"][h].to(torch.float64)
    top = torch.topk(key, c["top_k"], dim=1).indices
    return top, torch.softmax(torch.gather(sc, 1, top), dim=1)


def _router_grad64(c, s, R, idx, gate, dgate, h):
    """(dR, dW_router) of one head in 64 bits."""
    Ne = c["n_experts"]
    dS = gate * (dgate - (gate * dgate).sum(1, keepdim=True))
    dense = torch.zeros((R.shape[0], Ne), dtype=torch.float64, device="cuda")
    dense.scatter_(1, idx, dS)
    return dense @ s["W_router"][h].to(torch.float64), dense.t() @ R


def exact(case, seed):
    c = case
    T, Nh, dh, Ne, k, dff = _shape(c)
    f64 = torch.float64
    s = _inputs(c, seed)

    def heads(parts):
        """Per-head (T, ...) results to (T, n_heads, ...)."""
        return torch.stack(parts, 1)

    if c["path"] in ("forward", "train"):
        Ys, gates, dXs, dWrs, dWs = [], [], [], [], []
        for h in range(Nh):
            X = s["X"][:, h].to(f64)
            idx, gate = _route64(c, s, X, h)
            if c["path"] == "forward":
                Ys.append(_experts64(c, s, X, idx, gate, h))
            else:
                Y, dX, dgate, dW = _experts64(c, s, X, idx, gate, h, s["dY"][:, h].to(f64))
                dR, dWr = _router_grad64(c, s, X, idx, gate, dgate, h)
                Ys.append(Y)
                dXs.append(dX + dR)
                dWrs.append(dWr)
                dWs.append([None if w is None else w.float() for w in dW])
            gates.append(gate)
        out = [heads(Ys), None, heads(gates), None]
        if c["path"] == "train":
            out += [heads(dXs), torch.stack(dWrs)]
            out += [torch.stack([w[i] for w in dWs]) for i in range(3) if dWs[0][i] is not None]
        return out
    if c["path"] == "backward":
        dXs, dWrs, dWs = [], [], []
        for h in range(Nh):
            X = s["X"][:, h].to(f64)
            idx, gate = s["idx"][:, h].long(), s["gate"][:, h].to(f64)
            _, dX, dgate, dW = _experts64(c, s, X, idx, gate, h, s["dY"][:, h].to(f64))
            dR, dWr = _router_grad64(c, s, X, idx, gate, dgate, h)
            dXs.append(dX + dR)
            dWrs.append(dWr)
            dWs.append(dW)
        return [heads(dXs), torch.stack(dWrs)] + [
            torch.stack([w[i] for w in dWs]) for i in range(3) if dWs[0][i] is not None]
    if c["path"] == "routing":
        gates, dXs, dWrs = [], [], []
        for h in range(Nh):
            X = s["X"][:, h].to(f64)
            idx, gate = _route64(c, s, X, h)
            dX, dWr = _router_grad64(c, s, X, idx, gate, s["dgate"][:, h].to(f64), h)
            gates.append(gate)
            dXs.append(dX)
            dWrs.append(dWr)
        return [None, heads(gates), None, heads(dXs), torch.stack(dWrs)]
    dt = _torch_dtype(c)
    N = Nh * dh
    x, W_in, W_out = s["x"].to(f64), s["W_in"].to(f64), s["W_out"].to(f64)
    if c["path"] == "latent":
        # the router decides on the latent sub-tokens in the path's dtype
        lat = (x @ W_in.t()).to(dt).reshape(T, 2 * Nh, dh)
        Ys, gates = [], []
        for h in range(Nh):
            idx, gate = _route64(c, s, lat[:, Nh + h].to(f64), h)
            Ys.append(_experts64(c, s, lat[:, h].to(f64), idx, gate, h))
            gates.append(gate)
        Y = heads(Ys)
        full = (x @ W_in.t()).reshape(T, 2 * Nh, dh)
        return [Y.reshape(T, N) @ W_out.t(), full[:, :Nh], full[:, Nh:], Y, None, heads(gates),
                None]
    dout = s["dout"].to(f64)
    dY = (dout @ W_out).reshape(T, Nh, dh)
    dXs, dRs, dWrs, dWs = [], [], [], []
    for h in range(Nh):
        idx, gate = s["idx"][:, h].long(), s["gate"][:, h].to(f64)
        _, dX, dgate, dW = _experts64(c, s, s["X_lat"][:, h].to(f64), idx, gate, h, dY[:, h])
        dR, dWr = _router_grad64(c, s, s["R_lat"][:, h].to(f64), idx, gate, dgate, h)
        dXs.append(dX)
        dRs.append(dR)
        dWrs.append(dWr)
        dWs.append(dW)
    dlat = torch.cat([heads(dXs).reshape(T, N), heads(dRs).reshape(T, N)], 1)
    return ([dlat @ W_in, dlat.t() @ x, torch.stack(dWrs)]
            + [torch.stack([w[i] for w in dWs]) for i in range(3) if dWs[0][i] is not None]
            + [dout.t() @ s["Y_lat"].reshape(T, N).to(f64)])
