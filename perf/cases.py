"""Timed cases of the action-expert library: what a serving program has it do.

Each case is one call (or, for "cycle", the two calls of one control cycle)
through ``ActionExpert``: a joint denoising step, a whole per-token schedule, a
schedule from host budgets with finished environments skipped, or a new
observation (prefix K/V) followed by an urgency-aware release.  Batch 1 is one
robot, where launches and latency count; 8 to 64 environments are a fleet or a
simulator served by one GPU, where the matrix products count.  Weights are
random at the shapes of the bundled workloads; a fewer-layer expert stands for
the same layers of the full one, with less rounding carried from layer to layer.

``exact`` evaluates the same inputs in float64 with plain torch.
"""
import math
import random

import torch

import paper_2609_37772_amd as U


class Shape:
    """Model dimensions as ``uad_create`` reads them."""

    def __init__(self, n_layers, d_model, n_heads, n_kv_heads, head_dim, d_ff, action_dim, conditioning="input"):
        self.n_layers, self.d_model, self.n_heads, self.n_kv_heads = n_layers, d_model, n_heads, n_kv_heads
        self.head_dim, self.d_ff, self.action_dim = head_dim, d_ff, action_dim
        self.conditioning, self.rms_eps = conditioning, 1e-6


# width, query heads, KV heads, head dim, MLP width, conditioning, full depth
MODELS = {
    "tiny": (256, 4, 4, 64, 1024, "input", 2),
    "pi0": (1024, 8, 1, 256, 4096, "input", 18),
    "pi05": (1024, 8, 1, 256, 4096, "adarms", 18),
    "large": (1536, 12, 2, 128, 6144, "input", 24),
}


def shape_of(case):
    d, hq, hkv, hd, f, cond, _ = MODELS[case["model"]]
    return Shape(case["layers"], d, hq, hkv, hd, f, case["actions"], cond)


def _case(name, entry, model, layers, batch, chunk, prefix, budgets, actions=32, dtype="bf16", **more):
    return dict(name=name, entry=entry, model=model, layers=layers, batch=batch, chunk=chunk, prefix=prefix,
                budgets=budgets, actions=actions, dtype=dtype, **more)


def listed():
    return [
        # the smallest call: one step of the small fp32-weight expert, launch latency only
        _case("tiny_step", "step", "tiny", 2, 1, 16, 64, "uniform 10", actions=7, dtype="f32"),
        # one robot, one chunk: ten uniform steps from noise
        _case("pi0_b1_schedule", "schedule", "pi0", 18, 1, 50, 816, "uniform 10"),
        # one robot, one control cycle: a new observation's prefix, then the urgent
        # actions after one step, ghosts, the corrected tail (U = 5, K = 1, N* = 7, S = 10)
        _case("pi0_b1_cycle", "cycle", "pi0", 18, 1, 50, 816, "release 5 1 7 10"),
        # one robot, the adaptive-norm expert, per-token budgets in three groups
        _case("pi05_b1_schedule", "schedule", "pi05", 18, 1, 50, 816, "groups"),
        # a few robots with an odd chunk, prefix and action count
        _case("pi0_b3_ragged_step", "step", "pi0", 18, 3, 37, 501, "random", actions=7),
        # one GPU's share of a fleet over eight GPUs
        _case("pi0_b8_step", "step", "pi0", 18, 8, 50, 816, "random"),
        # new observations of 16 robots, fp32 prefix, then their release
        _case("pi0_b16_cycle", "cycle", "pi0", 6, 16, 50, 816, "release 3 1 3 10", dtype="f32"),
        # a half-size fleet: the later steps of a schedule whose environments finish
        _case("pi0_b32_step", "step", "pi0", 6, 32, 50, 816, "random"),
        # the fleet: one joint step over 64 environments
        _case("pi0_b64_step", "step", "pi0", 18, 64, 50, 816, "random"),
        # the fleet's whole chunk from its budgets, finished environments skipped
        _case("pi0_b64_budgets", "budgets", "pi0", 18, 64, 50, 816, "random"),
        # the fleet with the adaptive-norm expert
        _case("pi05_b64_step", "step", "pi05", 6, 64, 50, 816, "random"),
        # the wide expert with long chunks
        _case("large_b16_step", "step", "large", 8, 16, 128, 1024, "linear"),
    ]


def draw(rng):
    """One more case: any model and entry, batch 1 to 64, odd chunks, prefixes and action counts."""
    model = rng.choice(["tiny", "pi0", "pi0", "pi05", "large"])
    batch = int(round(2 ** rng.uniform(0, 6)))
    if model == "large":
        batch, chunk = max(1, batch // 4), rng.randint(24, 128)
    else:
        chunk = rng.randint(10, 64)
    layers = rng.randint(2, 6)
    if model == "pi0" and batch == 1:
        layers = 18
    entry = rng.choice(["step", "step", "schedule", "budgets", "cycle"])
    prefix = rng.randint(64, 1024)
    budgets = rng.choice(["uniform 10", "random", "linear"])
    if entry == "cycle":
        batch = min(batch, 16)
        n = rng.randint(2, 7)
        s = rng.randint(4, 10)
        budgets = "release %d %d %d %d" % (rng.randint(1, min(s - 1, 6)), rng.randint(1, n - 1), n, s)
    return dict(entry=entry, model=model, layers=layers, batch=batch, chunk=chunk, prefix=prefix, budgets=budgets,
                actions=rng.choice([7, 14, 32]), dtype=rng.choice(["bf16", "bf16", "f32"]))


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------
def budgets_of(case):
    """Per-token step budgets [batch][chunk], from the case alone."""
    B, H, kind = case["batch"], case["chunk"], case["budgets"].split()
    if kind[0] == "uniform":
        return [[int(kind[1])] * H for _ in range(B)]
    if kind[0] == "groups":  # 4 steps for the first tenth, 7 up to the half, 10 beyond
        return [[4 if 10 * i < H else 7 if 2 * i < H else 10 for i in range(H)] for _ in range(B)]
    if kind[0] == "linear":  # 3 to 12 along the chunk
        return [[3 + (18 * i + H - 1) // (2 * (H - 1)) for i in range(H)] for _ in range(B)]
    if kind[0] == "random":  # an urgent prefix on fewer steps than the tail, other ones per environment
        r, out = random.Random(20 * B + H), []
        for _ in range(B):
            u, n = r.randint(3, 10), r.randint(4, 10)
            k = r.randint(3, n - 1)
            out.append([k] * min(u, H) + [n] * (H - min(u, H)))
        return out
    raise ValueError(case["budgets"])


def tables_of(budgets):
    """Flow times, steps and masks of every joint step, as float32 / bool rows on the CPU."""
    n = torch.tensor(budgets, dtype=torch.float32)
    t, dt, mask = [], [], []
    for k in range(int(n.max())):
        t.append((n - torch.clamp(n, max=float(k))) / n)
        dt.append(torch.where(n > k, -(1.0 / n), torch.zeros_like(n)))
        mask.append(n <= k)
    return torch.stack(t), torch.stack(dt), torch.stack(mask)


def release_of(case):
    return [int(v) for v in case["budgets"].split()[1:]]


def _weights(case, g):
    s = shape_of(case)
    d, f, da, q, kv = s.d_model, s.d_ff, s.action_dim, s.n_heads * s.head_dim, s.n_kv_heads * s.head_dim
    ada = s.conditioning == "adarms"
    specs = [("action_in.w", (d, da)), ("action_in.b", (d,)), ("time_mlp_in.w", (d, d if ada else 2 * d)),
             ("time_mlp_in.b", (d,)), ("time_mlp_out.w", (d, d)), ("time_mlp_out.b", (d,))]
    for l in range(s.n_layers):
        p = "layers.%d." % l
        for norm in ("attn", "mlp"):
            if ada:
                specs += [(p + norm + "_mod.w", (3 * d, d)), (p + norm + "_mod.b", (3 * d,))]
            else:
                specs += [(p + norm + "_norm", (d,))]
        specs += [(p + "wq", (q, d)), (p + "wk", (kv, d)), (p + "wv", (kv, d)), (p + "wo", (d, q)),
                  (p + "w_gate", (f, d)), (p + "w_up", (f, d)), (p + "w_down", (d, f))]
    specs += [("final_mod.w", (2 * d, d)), ("final_mod.b", (2 * d,))] if ada else [("final_norm", (d,))]
    specs += [("action_out.w", (da, d)), ("action_out.b", (da,))]
    out = {}
    for name, shape in specs:
        w = torch.randn(shape, generator=g, device="cuda") * 0.02
        if name.endswith("_norm"):
            w += 1.0
        out[name] = w if case["dtype"] == "f32" else w.to(torch.bfloat16)
    return out


def inputs(case, seed):
    """(weights, prefix K, prefix V, initial noise) on the GPU."""
    s = shape_of(case)
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    weights = _weights(case, g)
    shape = (s.n_layers, case["batch"], case["prefix"], s.n_kv_heads, s.head_dim)
    kind = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    k, v = (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(kind) for _ in range(2))
    x0 = torch.randn((case["batch"], case["chunk"], s.action_dim), generator=g, device="cuda")
    return weights, k, v, x0


def _step_index(case):
    return min(2, max(max(row) for row in budgets_of(case)) - 1)


def prepare(case, seed):
    weights, k, v, x0 = inputs(case, seed)
    B, H, P, da = case["batch"], case["chunk"], case["prefix"], case["actions"]
    expert = U.ActionExpert(shape_of(case), B, H, P)
    expert.load_weights(weights)
    state = {"case": case, "expert": expert, "x0": x0, "x": torch.empty_like(x0)}
    if case["entry"] == "cycle":
        u, _, _, s = release_of(case)
        state.update(k=k, v=v, urgent=torch.empty((B, u, da), device="cuda"),
                     executed=torch.empty((B, s, da), device="cuda"), host=torch.empty((B, u, da), pin_memory=True))
        return state
    expert.set_prefix_kv(k, v, B, P)
    if case["entry"] == "budgets":
        state["budgets"] = torch.tensor(budgets_of(case), dtype=torch.int32).numpy()
    else:
        t, dt, mask = (a.cuda() for a in tables_of(budgets_of(case)))
        state.update(t=t, dt=dt, mask=mask.to(torch.uint8))
    if case["entry"] == "step":
        at = _step_index(case)
        state.update({n: state[n][at].contiguous() for n in ("t", "dt", "mask")}, velocity=torch.empty_like(x0))
    else:
        state.update(released=torch.zeros_like(x0), steps=torch.full((B, H), -1, dtype=torch.int32, device="cuda"))
    return state


def run(state):
    expert, entry, x = state["expert"], state["case"]["entry"], state["x"]
    x.copy_(state["x0"])  # a chunk starts from noise
    if entry == "step":
        expert.step(x, state["t"], state["dt"], state["mask"], state["velocity"])
        return {"x": x, "velocity": state["velocity"]}
    if entry == "cycle":
        u, k, n, s = release_of(state["case"])
        expert.set_prefix_kv(state["k"], state["v"], state["case"]["batch"], state["case"]["prefix"])
        expert.release(x, u, k, n, s, urgent=state["urgent"], executed=state["executed"], urgent_host=state["host"])
        return {"x": x, "urgent": state["urgent"], "executed": state["executed"], "host": state["host"]}
    if entry == "schedule":
        expert.schedule(x, state["t"], state["dt"], state["mask"], state["released"], state["steps"])
    else:
        expert.schedule_budgets(x, state["budgets"], state["released"], state["steps"])
    return {"x": x, "released": state["released"], "steps": state["steps"]}


# ----------------------------------------------------------------------------
# What a pass cannot do without, and how far two correct ones may differ
# ----------------------------------------------------------------------------
def work(case):
    """Weights once per joint step (they exceed the chip's caches), the prefix K/V of the evaluated
    environments per step, states in and out; the products of the evaluated environments' tokens."""
    s, H, P, B = shape_of(case), case["chunk"], case["prefix"], case["batch"]
    d, f, q, kv = s.d_model, s.d_ff, s.n_heads * s.head_dim, s.n_kv_heads * s.head_dim
    ada = s.conditioning == "adarms"
    layer = d * (q + 2 * kv) + q * d + 3 * d * f
    per_token = s.n_layers * layer + (d * d if ada else 3 * d * d) + 2 * s.action_dim * d
    mod = (6 * s.n_layers + 2) * d * d + 2 * d * d if ada else 0  # modulations and time MLP of one flow time
    attn = 4 * s.n_layers * q * H * (P + H)
    prefix = 2 * s.n_layers * P * kv
    if case["entry"] == "step":
        envs, times = [B], [len({t for t in tables_of(budgets_of(case))[0][_step_index(case)].flatten().tolist()})]
    elif case["entry"] == "cycle":
        n = release_of(case)[2]
        envs, times = [B] * n, [1] * n
    else:
        most = [max(row) for row in budgets_of(case)]
        envs = [sum(m > k for m in most) if case["entry"] == "budgets" and not ada else B for k in range(max(most))]
        times = [len(set(row.flatten().tolist())) for row in tables_of(budgets_of(case))[0]]
    total = {"bytes": 0.0, "flops": 0.0}
    for b, n in zip(envs, times):
        total["bytes"] += 2 * (per_token + mod) + 2 * b * prefix + 8 * b * H * s.action_dim
        total["flops"] += 2 * b * H * per_token + b * attn + 2 * n * mod
    if case["entry"] == "cycle":  # the new prefix in, its store out
        total["bytes"] += B * prefix * ((4 if case["dtype"] == "f32" else 2) + 2)
    return total


def tolerance(case):
    """fp16 projection operands, bf16 q / k / v and probabilities: two correct passes differ by 2e-3 to
    3e-3 (2-norm) in velocities, less in states."""
    return {"rel": 1e-2, "max": 0.1}


# ----------------------------------------------------------------------------
# The same in float64
# ----------------------------------------------------------------------------
def _rms(h):
    return h / torch.sqrt((h * h).mean(-1, keepdim=True) + 1e-6)


def _gelu(z):
    return 0.5 * z * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (z + 0.044715 * z ** 3)))


class Exact:
    """The expert in float64: x [B][H][Da], t [B][H] -> velocity."""

    def __init__(self, case, weights, k, v):
        self.s, self.case = shape_of(case), case
        # projections and prefix are bf16 by contract; norms, biases and action projections fp32
        self.w = {n: (w.to(torch.bfloat16) if w.dim() == 2 and not n.startswith("action") else w)
                  for n, w in weights.items()}
        self.k, self.v = k.to(torch.bfloat16), v.to(torch.bfloat16)

    def lin(self, x, name):
        return x @ self.w[name].double().t().contiguous()

    def attend(self, l, n):
        s = self.s
        B, H, p = n.shape[0], n.shape[1], "layers.%d." % l
        G = s.n_heads // s.n_kv_heads
        q = self.lin(n, p + "wq").view(B, H, s.n_kv_heads, G, s.head_dim).permute(0, 2, 3, 1, 4)
        q = q.reshape(B, s.n_kv_heads, G * H, s.head_dim).contiguous()
        kc, vc = (self.lin(n, p + m).view(B, H, s.n_kv_heads, s.head_dim) for m in ("wk", "wv"))
        k = torch.cat([self.k[l].double(), kc], 1).permute(0, 2, 3, 1).contiguous()
        v = torch.cat([self.v[l].double(), vc], 1).permute(0, 2, 1, 3).contiguous()
        o = torch.matmul(torch.softmax(torch.matmul(q, k) / math.sqrt(s.head_dim), -1), v)
        o = o.view(B, s.n_kv_heads, G, H, s.head_dim).permute(0, 3, 1, 2, 4).reshape(B, H, s.n_heads * s.head_dim)
        return self.lin(o.contiguous(), p + "wo")

    def mlp(self, l, n):
        p = "layers.%d." % l
        return self.lin(_gelu(self.lin(n, p + "w_gate")) * self.lin(n, p + "w_up"), p + "w_down")

    def __call__(self, x, t):
        s, w, d = self.s, self.w, self.s.d_model
        silu = torch.nn.functional.silu
        j = torch.arange(d // 2, dtype=torch.float64, device=x.device)
        arg = t.double()[..., None] * (1000.0 * 10000.0 ** (-j / (d // 2))).float().double()
        e = torch.cat([torch.sin(arg), torch.cos(arg)], -1)
        a = self.lin(x, "action_in.w") + w["action_in.b"].double()
        ada = s.conditioning == "adarms"
        u = silu(self.lin(e if ada else torch.cat([a, e], -1), "time_mlp_in.w") + w["time_mlp_in.b"].double())
        u = self.lin(u, "time_mlp_out.w") + w["time_mlp_out.b"].double()
        if not ada:
            h = u
            for l in range(s.n_layers):
                h = h + self.attend(l, _rms(h) * w["layers.%d.attn_norm" % l].double())
                h = h + self.mlp(l, _rms(h) * w["layers.%d.mlp_norm" % l].double())
            n = _rms(h) * w["final_norm"].double()
        else:
            c, h = silu(u), a

            def mods(name, parts):
                return (self.lin(c, name + ".w") + w[name + ".b"].double()).split(d, -1)[:parts]
            for l in range(s.n_layers):
                sc, sh, gate = mods("layers.%d.attn_mod" % l, 3)
                h = h + gate * self.attend(l, _rms(h) * (1.0 + sc) + sh)
                sc, sh, gate = mods("layers.%d.mlp_mod" % l, 3)
                h = h + gate * self.mlp(l, _rms(h) * (1.0 + sc) + sh)
            sc, sh = mods("final_mod", 2)
            n = _rms(h) * (1.0 + sc) + sh
        return self.lin(n, "action_out.w") + w["action_out.b"].double()


def exact(case, seed):
    weights, k, v, x0 = inputs(case, seed)
    f = Exact(case, weights, k, v)
    x = x0.double()
    if case["entry"] == "cycle":
        u, K, n, S = release_of(case)
        urgent_t = torch.ones_like(x0[..., 0])
        vsum = 0.0
        for i in range(n):
            uni = torch.full_like(urgent_t, (n - i) / n)
            t, step = uni, torch.full_like(uni, 1.0 / n)
            if i < K:
                t, step = uni.clone(), step.clone()
                t[:, :u], step[:, :u] = (K - i) / K, 1.0 / K
            vel = f(x, t)
            x = x - step.double()[..., None] * vel
            if i < K:
                vsum = vsum + vel[:, :u]
            if i == K - 1:
                urgent = x[:, :u].clone()
                x[:, :u] = x0[:, :u].double() - vsum / n
        shift = (x[:, :u] - urgent).sum(1, keepdim=True) / (S - u)
        return {"x": x, "urgent": urgent, "executed": torch.cat([urgent, x[:, u:S] + shift], 1), "host": urgent.cpu()}
    budgets = budgets_of(case)
    t, dt, mask = (a.cuda() for a in tables_of(budgets))
    if case["entry"] == "step":
        at = _step_index(case)
        vel = f(x, t[at])
        return {"x": torch.where(mask[at][..., None], x, x + dt[at].double()[..., None] * vel), "velocity": vel}
    last = torch.tensor(budgets, device=x.device) - 1
    released = torch.zeros_like(x)
    for i in range(t.shape[0]):
        x = torch.where(mask[i][..., None], x, x + dt[i].double()[..., None] * f(x, t[i]))
        released = torch.where((last == i)[..., None], x, released)
    return {"x": x, "released": released, "steps": None}
