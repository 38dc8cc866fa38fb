"""The work that is timed: what a program around the Topological Synapse has the library do, through its public calls.

Three kinds of callers share the library (see include/ws_synapse.h).  The producer turns a context into landmarks: density over
the cached keys (or the attention-mass proxy of it), the greedy selection, the gather.  The side agents attend over the landmarks
at every token they decode.  The main agent keeps the cache and its density current while it decodes: it gates the agents'
thoughts, injects the rows of an accepted one and refreshes the density.  The sizes are those of the workloads in
paper_2601_01298_amd/synthetic.py, the clouds follow its recipes (drawn on the GPU here), and draw() spreads over the range
between them: one head of a few hundred keys up to 24 layers of 16 heads with 32768 keys, or contexts of 131072 keys.

Every program here keeps its workspaces and output buffers, as bench.py and a serving loop do.
"""
import math

import torch

from paper_2601_01298_amd import binding as ws

HEAD_DIMS = (64, 128)
HIDDEN = 896          # width of the hidden states the gate compares
THETA = 0.5           # threshold of the gate
ROPE_BASE = 1.0e6


def listed():
    return [
        # the smallest use: one fp32 head of a few hundred keys through the whole path; launches and latency count
        dict(name="pass_tiny", kind="pass", cloud="mixture", dtype="f32", H=1, g=1, d=64, L=512, k=10, N=4),
        # one layer of a short context: a producer that refreshes layer by layer
        dict(name="density_layer", kind="density", cloud="scaled", dtype="bf16", H=16, d=64, L=4096),
        # all 24 layers of a 32k context in one call: the headline workload's density
        dict(name="density_headline", kind="density", cloud="drift", dtype="bf16", H=384, d=64, L=32768),
        # long context, few KV heads of dimension 128
        dict(name="density_long", kind="density", cloud="heavy", dtype="bf16", H=8, d=128, L=131072),
        # the selection at the same three scales, and on the layer with outliers whose far point moves at most steps
        dict(name="select_layer", kind="select", cloud="scaled", dtype="bf16", H=16, d=64, L=4096, k=82),
        dict(name="select_headline", kind="select", cloud="drift", dtype="bf16", H=384, d=64, L=32768, k=655),
        dict(name="select_outliers", kind="select", cloud="outliers", dtype="bf16", H=32, d=128, L=8192, k=164),
        dict(name="select_long", kind="select", cloud="heavy", dtype="bf16", H=8, d=128, L=131072, k=2621),
        # one token of 100 side agents over the synapse of all 24 layers: the call made at every decoded token
        dict(name="agents_headline", kind="agents", dtype="bf16", H=384, g=1, d=64, L=32768, k=655, N=100, form="synapse"),
        # a synapse filled and read once by a thousand agents
        dict(name="agents_many", kind="agents", dtype="bf16", H=32, g=1, d=128, L=8192, k=164, N=1000, form="gather"),
        # one decode step of the main agent: 100 thoughts gated, a thought's 8 rows injected, the density refreshed
        dict(name="upkeep_headline", kind="upkeep", cloud="drift", dtype="bf16", H=384, d=64, L=32768, m=8, N=100),
        # the attention-mass proxy over a long context with grouped query heads
        dict(name="mass_long", kind="mass", cloud="heavy", dtype="bf16", G=1, H=8, g=4, d=128, L=131072),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("pass", "density", "density", "select", "select", "select", "agents", "agents", "upkeep", "mass"))
    d = rng.choice(HEAD_DIMS)
    dtype = "f32" if rng.random() < 0.15 else "bf16"
    cloud = rng.choice(("mixture", "scaled", "drift", "outliers", "heavy"))
    wide = d * (4 if dtype == "f32" else 2)
    if kind == "pass":
        L = _log_int(rng, 200, 2000)
        return dict(kind=kind, cloud=cloud, dtype=dtype, H=rng.randint(1, 2), g=rng.choice((1, 2, 4)), d=d, L=L,
                    k=max(4, round(0.02 * L * rng.uniform(0.5, 1.5))), N=_log_int(rng, 1, 64))
    if kind in ("density", "select"):
        L = _log_int(rng, 300, 131072 if dtype == "bf16" else 16384)
        # no more than the headline's pairs (fp32 products run at a sixteenth of the bf16 rate) or its keys
        most = min(384 * 32768 ** 2 * 64 // d // (16 if dtype == "f32" else 1) // L ** 2, 384 * 32768 * 128 // wide // L)
        H = _log_int(rng, 1, max(1, min(384, most // 2)))
        if kind == "density":
            return dict(kind=kind, cloud=cloud, dtype=dtype, H=H, d=d, L=L)
        k = max(4, round(0.02 * L * rng.uniform(0.5, 1.5)))
        return dict(kind=kind, cloud=cloud, dtype=dtype, H=H, d=d, L=L, k=min(k, 2700))
    if kind == "agents":
        k = _log_int(rng, 10, 2700)
        L = min(131072, 50 * k + rng.randint(0, 49))
        H = _log_int(rng, 1, max(1, min(384, 384 * 32768 * 128 // wide // L)))
        g = rng.choice((1, 1, 2, 4, 8))
        N = _log_int(rng, 1, 1000 if dtype == "bf16" else 100)
        return dict(kind=kind, dtype=dtype, H=H, g=g, d=d, L=L, k=k, N=max(1, min(N, 2 ** 22 // (H * g * max(1, k // 256)))),
                    form=rng.choice(("synapse", "synapse", "gather", "indexed")))
    L = _log_int(rng, 500, 131072)
    H = _log_int(rng, 1, max(1, min(384, 384 * 32768 * 128 // wide // L)))
    if kind == "upkeep":
        return dict(kind=kind, cloud=cloud, dtype=dtype, H=H, d=d, L=L, m=rng.choice((1, 1, 2, 4, 8, 16)),
                    N=_log_int(rng, 1, 1000))
    G = max(1, H // 16) if H > 16 else 1
    return dict(kind="mass", cloud=cloud, dtype=dtype, G=G, H=H // G * G, g=rng.choice((1, 2, 4)), d=d, L=L)


# ---- inputs ---------------------------------------------------------------------------------------------------------------
def _torch_dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _generator(seed, tensor):
    gen = torch.Generator(device="cuda")
    gen.manual_seed((int(seed) * 8 + tensor) % (2 ** 62))
    return gen


def _cloud_chunk(kind, H, L, d, gen):
    """[H,L,d] fp32 rows of H heads: the recipes of synthetic.py."""
    dev = "cuda"

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev)

    if kind == "heavy":
        # anisotropic (eigenvalues ~ 1/j) and heavy-tailed (Student-t, 3 degrees of freedom)
        lam = 1.0 / torch.arange(1, d + 1, device=dev, dtype=torch.float32)
        lam *= d / lam.sum()
        U = torch.linalg.qr(normal(H, d, d))[0]
        chi = normal(H, L, d).square_()
        chi += normal(H, L, d).square_()
        chi += normal(H, L, d).square_()
        x = normal(H, L, d) / (chi / 3.0).sqrt_()
        return torch.matmul(x * lam.sqrt(), U.transpose(1, 2).contiguous())
    comps = {"mixture": 8, "scaled": 32, "drift": 64, "outliers": 128}[kind]
    centres = 2.0 * normal(H, comps, d)
    assign = torch.randint(0, comps, (H, L), generator=gen, device=dev)
    x = torch.gather(centres, 1, assign[:, :, None].expand(H, L, d)).add_(normal(H, L, d), alpha=0.5)
    if kind == "scaled":
        x *= torch.rand((H, 1, d), generator=gen, device=dev) * 1.5 + 0.5
    elif kind == "drift":
        x.add_(torch.cumsum(normal(H, L, d), dim=1), alpha=0.02)
    elif kind == "outliers":
        far = torch.rand((H, L), generator=gen, device=dev) < 0.01
        x = torch.where(far[:, :, None], torch.rand((H, L, d), generator=gen, device=dev) * 16.0 - 8.0, x)
    return x


def _cloud(case, seed, tensor, rows=None):
    """[H,L,d] keys (tensor 0) or values (tensor 1), a few heads at a time."""
    H, L, d = case["H"], rows or case["L"], case["d"]
    gen = _generator(seed, tensor)
    out = torch.empty((H, L, d), dtype=_torch_dtype(case), device="cuda")
    step = max(1, min(H, (1 << 27) // (L * d)))
    for h in range(0, H, step):
        n = min(step, H - h)
        out[h:h + n] = _cloud_chunk(case.get("cloud", "mixture"), n, L, d, gen)
    return out


def _bandwidth(K):
    """sigma^2 = tr(Cov)/16 per head, as host floats."""
    var = [K[h].float().var(dim=0, unbiased=False).sum() for h in range(K.shape[0])]
    return (torch.stack(var) / 16.0).sqrt().tolist()


def _density_estimate(K, sigma, gen):
    """[H,L] density against 64 sampled keys of the head, self term included: what the selection is handed, made without
    the library so that the selection alone is what its cases time."""
    H, L, d = K.shape
    m = min(64, L)
    rho = torch.empty((H, L), dtype=torch.float32, device="cuda")
    for h in range(H):
        x = K[h].float()
        pick = torch.randint(0, L, (m,), generator=gen, device="cuda")
        s = x[pick]
        d2 = (x.square().sum(1, keepdim=True) + s.square().sum(1)[None] - 2.0 * (x @ s.t().contiguous())).clamp_(min=0.0)
        w = torch.exp(d2 * (-0.5 / sigma[h] ** 2))
        w[pick, torch.arange(m, device="cuda")] = 0.0
        rho[h] = (1.0 + w.sum(1) * (L / m)) / L
    return rho


def _space(op, case, **kw):
    dt = ws.WS_F32 if case["dtype"] == "f32" else ws.WS_BF16
    n = ws.ws_synapse_workspace_bytes(op, dt, kw.pop("H", case["H"]), kw.pop("L", case.get("L", 1)), case["d"], **kw)
    return torch.empty(n, dtype=torch.uint8, device="cuda") if n else None


def _empty(shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    kind, H, d = case["kind"], case["H"], case["d"]
    dt = _torch_dtype(case)
    st = dict(case=case)

    def normal(shape, tensor):
        return torch.randn(shape, generator=_generator(seed, tensor), device="cuda").to(dt)

    if kind in ("density", "select", "pass", "mass"):
        st["K"] = _cloud(case, seed, 0)
    if kind in ("density", "pass"):
        st["sigma"] = _bandwidth(st["K"])
        st["rho"] = _empty((H, case["L"]))
        st["ws_density"] = _space(ws.WS_OP_DENSITY, case)
    if kind == "select":
        st["rho"] = _density_estimate(st["K"], _bandwidth(st["K"]), _generator(seed, 2))
    if kind in ("select", "pass"):
        st["idx"] = _empty((H, case["k"]), torch.int32)
        st["ws_select"] = _space(ws.WS_OP_SELECT, case, k=case["k"])
    if kind in ("pass", "agents"):
        k, N, Hq = case["k"], case["N"], H * case["g"]
        st["Q"] = normal((N, Hq, d), 3)
        st["O"] = _empty((N, Hq, d))
        st["ws_attend"] = _space(ws.WS_OP_ATTEND, case, L=1, k=k, N=N, Hq=Hq)
        st["Ks"], st["Vs"] = _empty((H, k, d), dt), _empty((H, k, d), dt)
    if kind == "pass":
        st["V"] = _cloud(case, seed, 1)
    if kind == "agents":
        L = case["L"]
        if case["form"] == "synapse":
            st["Ks"], st["Vs"] = _cloud(case, seed, 0, rows=k), _cloud(case, seed, 1, rows=k)
        else:
            st["K"], st["V"] = _cloud(case, seed, 0), _cloud(case, seed, 1)
            order = torch.rand((H, L), generator=_generator(seed, 4), device="cuda").argsort(dim=1)
            st["idx"] = order[:, :k].to(torch.int32).contiguous()
    if kind == "upkeep":
        m, N, L = case["m"], case["N"], case["L"]
        st["h"] = normal((HIDDEN,), 5)
        mix = torch.rand((N, 1), generator=_generator(seed, 6), device="cuda") * 3.5 - 0.5
        st["T"] = (mix * st["h"].float() + normal((N, HIDDEN), 7).float()).to(dt)
        st["Kc"], st["Vc"] = _cloud(case, seed, 0), _cloud(case, seed, 1)      # caches with room for exactly this thought
        st["Knew"], st["Vnew"] = normal((H, m, d), 8) * 2, normal((H, m, d), 9) * 2
        st["pos"] = torch.randint(0, 4 * L, (m,), generator=_generator(seed, 10), device="cuda").to(torch.int32)
        st["sigma"] = _bandwidth(st["Kc"])
        st["rho_old"] = torch.rand((H, L - m), generator=_generator(seed, 11), device="cuda") * 0.02 + 1.0 / L
        st["rho_new"] = _empty((H, L))
        st["score"], st["accept"] = _empty((N,)), _empty((N,), torch.int32)
        st["ws_inject"] = _space(ws.WS_OP_INJECT, case, k=m)
        st["ws_append"] = _space(ws.WS_OP_DENSITY_APPEND, case)
    if kind == "mass":
        Hq = H * case["g"]
        st["Q"] = normal((Hq, d), 3)
        st["out"] = _empty((H, case["L"]))
        st["ws_mass"] = _space(ws.WS_OP_ATTENTION_MASS, case, Hq=Hq)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "density":
        return ws.ws_synapse_density(st["K"], st["sigma"], rho=st["rho"], workspace=st["ws_density"])
    if kind == "select":
        # check=False: the serving loop reads the failure flag later, once for many calls
        return ws.ws_synapse_select(st["K"], st["rho"], case["k"], 0.5, idx=st["idx"], workspace=st["ws_select"], check=False)
    if kind == "pass":
        ws.ws_synapse_density(st["K"], st["sigma"], rho=st["rho"], workspace=st["ws_density"])
        ws.ws_synapse_select(st["K"], st["rho"], case["k"], 0.5, idx=st["idx"], workspace=st["ws_select"], check=False)
        ws.ws_synapse_gather(st["K"], st["V"], st["idx"], Ks=st["Ks"], Vs=st["Vs"])
        ws.ws_synapse_attend(st["Q"], st["Ks"], st["Vs"], O=st["O"], workspace=st["ws_attend"])
        return [st["rho"], st["idx"], st["Ks"], st["Vs"], st["O"]]
    if kind == "agents":
        if case["form"] == "indexed":
            return ws.ws_synapse_attend_indexed(st["Q"], st["K"], st["V"], st["idx"], O=st["O"], workspace=st["ws_attend"])
        if case["form"] == "gather":
            ws.ws_synapse_gather(st["K"], st["V"], st["idx"], Ks=st["Ks"], Vs=st["Vs"])
        ws.ws_synapse_attend(st["Q"], st["Ks"], st["Vs"], O=st["O"], workspace=st["ws_attend"])
        return [st["O"]] if case["form"] == "synapse" else [st["O"], st["Ks"], st["Vs"]]
    if kind == "upkeep":
        m, L = case["m"], case["L"]
        ws.ws_synapse_gate(st["h"], st["T"], THETA, score=st["score"], accept=st["accept"])
        ws.ws_synapse_inject(st["Kc"], st["Vc"], L - m, st["Knew"], st["Vnew"], st["pos"], ROPE_BASE, workspace=st["ws_inject"])
        ws.ws_synapse_density_append(st["Kc"], m, st["sigma"], st["rho_old"], rho_new=st["rho_new"], workspace=st["ws_append"])
        return [st["score"], st["accept"], st["Kc"], st["Vc"], st["rho_new"]]
    return ws.ws_synapse_attention_mass(st["K"], st["Q"], case["G"], out=st["out"], workspace=st["ws_mass"])


# ---- what a pass cannot do without ------------------------------------------------------------------------------------------
def work(case):
    kind, H, d = case["kind"], case["H"], case["d"]
    es = 4 if case["dtype"] == "f32" else 2
    nbytes = flops = 0.0
    if kind in ("density", "pass"):
        L = case["L"]
        nbytes += H * L * (d * es + 4)                  # keys in, densities out
        flops += H * L * L * d                          # every unordered pair once, 2 d flop
    if kind in ("select", "pass"):
        L, k = case["L"], case["k"]
        nbytes += H * (L * 4 + k * 4) + (H * L * d * es if kind == "select" else 0)
        flops += 3.0 * H * L * d                        # one distance per key at the very least
    if kind in ("agents", "pass"):
        k, N, Hq = case["k"], case["N"], H * case["g"]
        nbytes += 2 * H * k * d * es + N * Hq * d * (es + 4)
        if kind == "pass" or case["form"] == "gather":
            nbytes += 2 * H * k * d * es + H * k * 4
        flops += 4.0 * N * Hq * k * d
    if kind == "upkeep":
        m, N, L = case["m"], case["N"], case["L"]
        nbytes += (N + 1) * HIDDEN * es + 8 * N + 4 * H * m * d * es + H * L * (d * es + 8)
        flops += 6.0 * N * HIDDEN + 3.0 * H * L * m * d
    if kind == "mass":
        nbytes += H * case["L"] * (d * es + 4)
        flops += 2.0 * H * case["g"] * case["L"] * d
    return dict(bytes=float(nbytes), flops=float(flops))


def tolerance(case):
    """About four times what was measured: densities, attention, mass and refresh against the same sums in 64 bits, indices
    between the two selection kernels, which sum a distance in different orders.  Their picks differ only where two keys
    tie to fp32 rounding and swap places (at most 6e-4 of the picks, on the long context)."""
    kind = case["kind"]
    if kind == "select":
        return {"differ": 2.5e-3}
    if kind == "density":
        return {"rel": 2.5e-6, "max": 8e-6}             # measured 5.9e-7, 1.8e-6
    if kind == "mass":
        return {"rel": 2e-6, "max": 2.5e-5}             # measured 4.6e-7, 6.2e-6
    if kind == "upkeep":
        # the refreshed densities measured 2.7e-8; a rotated key may round to the neighbouring bf16 number
        return {"rel": 1e-5, "max": 8e-3, "differ": 2.5e-3}
    return {"rel": 4e-6, "max": 3e-5, "differ": 2.5e-3}     # attention: measured 9.6e-7, 6.7e-6


# ---- the outputs in 64 bits -------------------------------------------------------------------------------------------------
def _exact_density(X, sigma, rows=None):
    """Kernel sums of the given rows (all by default) of one head over all its keys, in 64 bits."""
    x = X.double()
    x = x - x.mean(dim=0)
    y = x if rows is None else x[rows]
    n = x.square().sum(1)
    out = torch.empty(y.shape[0], dtype=torch.float64, device=X.device)
    step = max(1, (1 << 27) // x.shape[0])
    for a in range(0, y.shape[0], step):
        e = (y[a:a + step] @ x.t().contiguous()).mul_(2.0).sub_(n[None]).sub_(y[a:a + step].square().sum(1)[:, None])
        out[a:a + step] = e.clamp_(max=0.0).mul_(0.5 / sigma ** 2).exp_().sum(1)
    return out


def _exact_attend(Q, Ks, Vs):
    N, Hq, d = Q.shape
    g = Hq // Ks.shape[0]
    out = torch.empty((N, Hq, d), dtype=torch.float64, device=Q.device)
    for q in range(Hq):
        z = (Q[:, q].double() @ Ks[q // g].double().t().contiguous()) / math.sqrt(d)
        out[:, q] = torch.softmax(z, dim=1) @ Vs[q // g].double()
    return out


def exact(case, seed):
    kind, H, d = case["kind"], case["H"], case["d"]
    if kind == "select" or (kind in ("density", "pass") and H * case["L"] ** 2 > 2 ** 38):
        return None                                         # picks have no value in 64 bits; the largest sweeps take too long
    st = prepare(case, seed)
    if kind in ("density", "pass"):
        rho = torch.stack([_exact_density(st["K"][h], st["sigma"][h]) for h in range(H)]) / case["L"]
        return rho if kind == "density" else [rho, None, None, None, None]
    if kind == "agents":
        if case["form"] == "synapse":
            return [_exact_attend(st["Q"], st["Ks"], st["Vs"])]
        at = st["idx"].long()[:, :, None].expand(-1, -1, d)
        Ks, Vs = st["K"].gather(1, at), st["V"].gather(1, at)
        O = _exact_attend(st["Q"], Ks, Vs)
        return O if case["form"] == "indexed" else [O, Ks.double(), Vs.double()]
    if kind == "upkeep":
        m, L = case["m"], case["L"]
        h, T = st["h"].double(), st["T"].double()
        score = (T @ h) / (h.norm() * T.norm(dim=1))
        ang = st["pos"].double()[:, None] * ROPE_BASE ** (-2.0 / d * torch.arange(d // 2, device="cuda", dtype=torch.float64))
        x0, x1 = st["Knew"].double().split(d // 2, dim=2)
        Kr = torch.cat([x0 * ang.cos() - x1 * ang.sin(), x1 * ang.cos() + x0 * ang.sin()], dim=2)
        Kc = st["Kc"]
        Kc[:, L - m:] = Kr.to(Kc.dtype)
        rho = torch.empty((H, L), dtype=torch.float64, device="cuda")
        for i in range(H):
            x, s = Kc[i].double(), st["sigma"][i]
            w = torch.stack([torch.exp((x - x[L - m + r]).square().sum(1) * (-0.5 / s ** 2)) for r in range(m)])
            rho[i, :L - m] = st["rho_old"][i].double() * (L - m) + w[:, :L - m].sum(0)
            rho[i, L - m:] = w.sum(1)
        return [score, None, None, None, rho / L]
    g, G = case["g"], case["G"]
    A = torch.zeros((G, case["L"]), dtype=torch.float64, device="cuda")
    for q in range(H * g):
        A[q // (H * g // G)] += torch.softmax(st["K"][q // g].double() @ st["Q"][q].double() / math.sqrt(d), dim=0)
    return (1.0 / A.clamp(min=1e-30)).repeat_interleave(H // G, dim=0)
