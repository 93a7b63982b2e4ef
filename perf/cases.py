"""The routed-attention calls that a user of this library has it do, as cases to be timed.

Every case is one context of `paper_2607_20125_amd.headcast` and one denoising step on it:

* ``step``      `append_block` of the current block (the overwrite that every denoising step
                makes) and `attention`, for each layer of the context;
* ``static``    the same through `attention_static`, the call for callers that cannot allocate;
* ``install``   `set_head_types` (restored labels, or a table decided offline) and the layer's
                first `attention`;
* ``classify``  the one-time `classify_heads` of a layer on a full window and its first routed
                `attention`.

Inputs are N(0, 1) in bf16, as the projections of normalised latents give them.  For
``classify`` the heads carry the structure that the method looks for (a shift towards block 0
or towards the current block, or a Gaussian of the distance on the frame), so that all four
labels come up.
"""
import math

import torch

from paper_2607_20125_amd import headcast as hc

SINK, DUMMY, SPATIAL, GLOBAL = hc.SINK, hc.DUMMY, hc.SPATIAL, hc.GLOBAL
THETA, THETA_SCORE, GAMMA = 0.95, 0.755, 5.0     # the library's defaults

# What a case holds unless it says otherwise: one layer of the 12-head, 128-dim model with three
# frames a block, a full window of seven blocks, radius 4 and proxy radius 2.
_BASE = dict(call="step", layers=1, heads=12, dim=128, frames=3, window=7, filled=7, radius=4,
             proxy=2, cell=0, sd=1)


def _case(name, gh, gw, mix, **more):
    sink, dummy, spatial, glob = mix
    c = dict(_BASE, name=name, gh=gh, gw=gw, sink=sink, dummy=dummy, spatial=spatial)
    c["global"] = glob
    c.update(more)
    return c


def listed():
    return [
        # the smallest context of the tests and of the smoke run: one head of each type, 128
        # tokens a block, where launches and latency are all there is
        _case("tiny_step", 8, 8, (1, 1, 1, 1), heads=4, dim=64, frames=2, window=4, filled=4, radius=1),
        # a small preview grid with 64-dim heads, four frames a block, rows that are not a
        # multiple of eight and a window that is not full yet
        _case("ragged_d64_step", 23, 46, (4, 4, 4, 4), heads=16, dim=64, frames=4, window=6, filled=5,
              radius=3),
        # a whole denoising step of the 30-layer 480P model, a different head table in each layer
        _case("model_480p", 30, 52, (90, 90, 90, 90), layers=30),
        # one average routed layer of the 720P model, the benchmark's default workload
        _case("step_720p", 45, 80, (2, 4, 4, 2)),
        # one average routed layer at 1080P, the largest grid
        _case("step_1080p", 68, 120, (2, 4, 4, 2)),
        # the fill phase: before the window is full every head is Global
        _case("fill_480p", 30, 52, (0, 0, 0, 12), filled=3),
        # a full-window layer at 720P: what a step costs without routing
        _case("full_720p", 45, 80, (0, 0, 0, 12)),
        # the one-time classification of a layer, then its first routed attention
        _case("classify_480p", 30, 52, (3, 3, 3, 3), call="classify"),
        _case("classify_720p", 45, 80, (2, 4, 4, 2), call="classify"),
        # the 10x10-cell form of the Spatial heads
        _case("cells_720p", 45, 80, (2, 4, 4, 2), cell=10),
        # two blocks for each Sink and Dummy head
        _case("two_block_480p", 30, 52, (3, 3, 3, 3), sd=2),
        # the call that allocates nothing, with as many Global heads as its scratch holds
        _case("static_480p", 30, 52, (3, 4, 2, 3), call="static"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: grids from 8x8 to 68x120, 1 to 4 frames, every call and option."""
    while True:
        call = rng.choice(["step"] * 6 + ["classify"] * 2 + ["static", "install"])
        gh = _log_int(rng, 8, 68)
        gw = max(8, min(120, int(round(gh * rng.uniform(1.0, 1.9)))))
        frames = rng.choice([1, 2, 3, 3, 3, 4])
        if frames * gh * gw % 8:
            continue
        heads = rng.choice([4, 8, 12, 12, 12, 16])
        window = rng.choice([4, 5, 6, 7, 7, 7, 8])
        filled = window if call == "classify" or rng.random() < 0.7 else rng.randint(1, window)
        kinds = [rng.choice([SINK, DUMMY, DUMMY, SPATIAL, SPATIAL, GLOBAL]) for _ in range(heads)]
        if rng.random() < 0.15:
            kinds = [GLOBAL] * heads
        c = _case("", gh, gw, [kinds.count(t) for t in (SINK, DUMMY, SPATIAL, GLOBAL)], call=call,
                  heads=heads, dim=rng.choice([64, 128, 128, 128]), frames=frames, window=window,
                  filled=filled, radius=rng.choice([1, 2, 3, 4, 4, 4, 5, 6]))
        option = rng.random()
        if option < 0.15 and call in ("step", "install"):
            c["cell"] = rng.choice([8, 10, 12])
        elif option < 0.3 and call != "classify":
            c["sd"] = 2
        slots = (c["global"] * c["filled"] + 2 * (c["sink"] + c["dummy"])) * (_tokens(c) // 128 + 1)
        if call == "static" and slots > 950:
            continue
        if work(c)["flops"] > 5e12:
            continue
        del c["name"]
        return c


def _tokens(c):
    return c["frames"] * c["gh"] * c["gw"]


def _tables(c):
    """Head types of every layer: the case's counts, spread over the layers in a fixed order."""
    flat = ([SINK] * c["sink"] + [DUMMY] * c["dummy"] + [SPATIAL] * c["spatial"] + [GLOBAL] * c["global"])
    g = torch.Generator()
    g.manual_seed(len(flat))
    order = torch.randperm(len(flat), generator=g).tolist()
    flat = [flat[i] for i in order]
    return [flat[i * c["heads"]:(i + 1) * c["heads"]] for i in range(c["layers"])]


def _current(c):
    return c["filled"] - 1


def _inputs(c, seed, layer, kinds):
    """Q of the current block, the window's K and V, and the K and V that this step appends."""
    H, L, d, n = c["heads"], _tokens(c), c["dim"], c["filled"]
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * int(seed) + layer)

    def normal(rows):
        return torch.randn((H, rows, d), generator=g, device="cuda")

    q, k, v = normal(L), normal(n * L), normal(n * L)
    if c["call"] == "classify":
        t = torch.arange(n * L, device="cuda")
        pos = t % (c["gh"] * c["gw"])
        y = (pos // c["gw"]).float() - c["gh"] // 2
        x = (pos % c["gw"]).float() - c["gw"] // 2
        r2 = -8.0 * (y * y + x * x)
        hi = r2.bfloat16().float()
        one, sixteen = torch.ones_like(y), torch.full_like(y, 16.0)
        for h, kind in enumerate(kinds):
            if kind in (SINK, DUMMY):        # three logits more on block 0 or on the current block
                u = torch.randn(d, generator=g, device="cuda")
                u /= u.norm()
                q[h] += math.sqrt(d) * u
                blk = 0 if kind == SINK else n - 1
                k[h, blk * L:(blk + 1) * L] += 3 * u
            elif kind == SPATIAL:            # -8 |p - p'|^2 / sqrt(d) on the logits
                k[h, :, :6] = torch.stack([16 * y, 16 * x, hi, r2 - hi, sixteen, sixteen], 1)
                lo = (r2 - hi) / 16
                q[h, :, :6] = torch.stack([y, x, one, one, hi / 16, lo], 1)[:L]
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    if c["call"] in ("classify", "install"):
        return q, k, v, None, None
    return q, k, v, normal(L).bfloat16(), normal(L).bfloat16()


def prepare(case, seed):
    cfg = hc.make_config(n_layers=case["layers"], n_heads=case["heads"], head_dim=case["dim"],
                         grid_h=case["gh"], grid_w=case["gw"], frames_per_block=case["frames"],
                         window_blocks=case["window"], spatial_radius=case["radius"],
                         proxy_radius=case["proxy"], spatial_cell=case["cell"], sd_blocks=case["sd"])
    ctx = hc.Context(cfg, 0)
    layers = []
    for i, kinds in enumerate(_tables(case)):
        q, k, v, kb, vb = _inputs(case, seed, i, kinds)
        o = torch.empty(q.shape, dtype=torch.float32, device="cuda")
        if case["call"] in ("step", "static"):
            ctx.set_head_types(i, kinds, _current(case), k, v)
            k = v = None
        layers.append((kinds, q, k, v, kb, vb, o))
    torch.cuda.synchronize()
    return dict(case=case, ctx=ctx, layers=layers)


def run(state):
    case, ctx = state["case"], state["ctx"]
    call, cur = case["call"], _current(case)
    outs = []
    for i, (kinds, q, k, v, kb, vb, o) in enumerate(state["layers"]):
        if call == "classify":
            kinds, stats = ctx.classify_heads(i, cur, q, k, v)
            outs += [kinds, stats]
        elif call == "install":
            ctx.set_head_types(i, kinds, cur, k, v)
        else:
            ctx.append_block(i, cur, kb, vb)
        if call == "static":
            ctx.attention_static(i, q, kinds, o)
        else:
            ctx.attention(i, q, kinds, o)
        outs.append(o)
    return outs


def _cells(n, size):
    """Edges of the cells along one axis: all `size` wide but the last, which ends at the border."""
    m = max(1, (2 * n + size) // (2 * size))
    return [i * size for i in range(m)] + [n]


def _axis_pairs(n, r):
    return sum(min(n - 1, i + r) - max(0, i - r) + 1 for i in range(n))


def _pairs(c, kind, radius=None):
    """(query, key) pairs of one head."""
    L, n, F = _tokens(c), c["filled"], c["frames"]
    if kind == GLOBAL:
        return L * n * L
    if kind in (SINK, DUMMY):
        return L * L * (min(n, 2) if c["sd"] == 2 else 1)
    if c["cell"] and radius is None:
        hs, ws = _cells(c["gh"], c["cell"]), _cells(c["gw"], c["cell"])
        area = sum((b - a) ** 2 for a, b in zip(hs, hs[1:])) * sum((b - a) ** 2 for a, b in zip(ws, ws[1:]))
    else:
        r = c["radius"] if radius is None else radius
        area = _axis_pairs(c["gh"], r) * _axis_pairs(c["gw"], r)
    return F * n * F * area


def work(case):
    L, d, H, n = _tokens(case), case["dim"], case["heads"], case["filled"]
    pairs, keys = 0, 0
    for kind, count in zip((SINK, DUMMY, SPATIAL, GLOBAL), (case["sink"], case["dummy"], case["spatial"], case["global"])):
        pairs += count * _pairs(case, kind)
        keys += count * (L * (min(n, 2) if case["sd"] == 2 else 1) if kind in (SINK, DUMMY) else n * L)
    heads = H * case["layers"]
    row = 2 * d                                  # bytes of a bf16 row
    # Q in, O out, and the keys and values that the heads attend to
    total = heads * L * row + heads * L * d * 4 + 2 * keys * row
    if case["call"] in ("classify", "install"):
        total += 2 * heads * n * L * row         # the window that is split
        if case["call"] == "classify":
            # O_ref over the window (O_sink and O_dummy are parts of it) and the Spatial proxy
            pairs += heads * (_pairs(case, GLOBAL) + _pairs(case, SPATIAL, case["proxy"]))
    else:
        total += 2 * 2 * heads * L * row         # the appended block in, and into the cache
    return {"bytes": total, "flops": 4 * d * pairs}


def tolerance(case):
    # probabilities are bf16 operands of the second product: 2^-9 each, and less in a mean over
    # many keys of random sign (1.7e-3 against 64 bits); `max` is of single elements over the
    # result's root mean square
    return {"rel": 7e-3, "max": 0.06}


def _attend(q, k, v, keep=None):
    """Softmax attention of one head in 64 bits; keep(rows) gives the mask of some rows."""
    k, v, q = k.double(), v.double(), q.double() / math.sqrt(q.shape[1])
    out = torch.empty_like(q)
    step = max(1, (1 << 28) // k.shape[0])
    for a in range(0, q.shape[0], step):
        s = q[a:a + step] @ k.t()
        if keep is not None:
            s.masked_fill_(~keep(torch.arange(a, min(a + step, q.shape[0]), device=q.device)), -math.inf)
        out[a:a + step] = torch.softmax(s, 1) @ v
    return out


def _spatial_mask(c, radius):
    n, P, gw = c["filled"], c["gh"] * c["gw"], c["gw"]
    pos = torch.arange(n * _tokens(c), device="cuda") % P
    ky, kx = pos // gw, pos % gw

    def window(rows):
        y, x = (rows % P // gw)[:, None], (rows % P % gw)[:, None]
        return ((ky - y).abs() <= radius) & ((kx - x).abs() <= radius)

    if not c["cell"]:
        return window

    def index(at, edges):
        return torch.bucketize(at, torch.tensor(edges[1:-1], device="cuda"), right=True)

    hs, ws = _cells(c["gh"], c["cell"]), _cells(c["gw"], c["cell"])
    kcell = index(ky, hs) * len(ws) + index(kx, ws)

    def cell(rows):
        return kcell == (index(rows % P // gw, hs) * len(ws) + index(rows % P % gw, ws))[:, None]
    return cell


def _routed(c, kinds, q, k, v):
    L, n = _tokens(c), c["filled"]
    out = []
    for h, kind in enumerate(kinds):
        blocks, keep = list(range(n)), None
        if kind == SINK:
            blocks = [0] if c["sd"] == 1 else [0, n - 1]
        elif kind == DUMMY:
            blocks = [n - 1] if c["sd"] == 1 else [n - 2, n - 1]
        elif kind == SPATIAL:
            keep = _spatial_mask(c, c["radius"])
        blocks = sorted({max(b, 0) for b in blocks})
        rows = torch.cat([torch.arange(b * L, (b + 1) * L, device="cuda") for b in blocks])
        out.append(_attend(q[h], k[h][rows], v[h][rows], keep))
    return torch.stack(out)


def _decide(stats):
    if stats[0] >= THETA:
        return SINK
    if stats[1] >= THETA:
        return DUMMY
    return SPATIAL if stats[2] >= THETA and stats[5] >= THETA_SCORE else GLOBAL


def _classified(c, q, k, v):
    L = _tokens(c)
    types, stats = [], []
    for h in range(c["heads"]):
        ref = _attend(q[h], k[h], v[h])
        sink = _attend(q[h], k[h, :L], v[h, :L])
        dummy = _attend(q[h], k[h, -L:], v[h, -L:])
        spatial = _attend(q[h], k[h], v[h], _spatial_mask(dict(c, cell=0), c["proxy"]))
        cos = [torch.nn.functional.cosine_similarity(o, ref, 1, 1e-30) for o in (sink, dummy, spatial)]
        p5 = torch.quantile(cos[2], 0.05)
        mse = ((spatial - ref) ** 2).mean()
        s = [cos[0].mean(), cos[1].mean(), cos[2].mean(), p5, mse, p5 - GAMMA * mse]
        stats.append([float(x) for x in s])
        types.append(_decide(stats[-1]))
    return types, stats


def exact(case, seed):
    outs = []
    for i, kinds in enumerate(_tables(case)):
        q, k, v, kb, vb = _inputs(case, seed, i, kinds)
        if case["call"] == "classify":
            kinds, stats = _classified(case, q, k, v)
            outs += [torch.tensor(kinds, dtype=torch.uint8), torch.tensor(stats, dtype=torch.float64)]
        elif kb is not None:
            L = _tokens(case)
            k, v = torch.cat([k[:, :-L], kb], 1), torch.cat([v[:, :-L], vb], 1)
        outs.append(_routed(case, kinds, q, k, v))
    return outs
