"""The work this framework is measured by: outer iterations of H-SADMM's consensus side on one GPU.

A case is a network (its conv / linear weight table), the sparsity constraint on it, the number R of replicas the node
averages, and the form of the step its program calls:

  step       hsadmm_project_compact + hsadmm_expand: averaging, candidate, selection, projection, dual update, shrinkage
             and recovery (the default step of the benchmark), dual updated in place, nothing known beforehand
  predicted  the same step from the second outer iteration on, at a settled support: hsadmm_step with the previous
             iteration's selection record and the dual written to a second buffer
  weighted   the full candidate of Eq. (9): hsadmm_project_weighted_compact + hsadmm_expand_dual
  norms      the same with the four residual norms the penalties and the stopping test need: hsadmm_step +
             hsadmm_retrain_expand
  retrain    an iteration after the masks are frozen, with its norms: hsadmm_retrain_project + hsadmm_retrain_expand
  union      the exchange with another node: hsadmm_mask_or, hsadmm_compact_sum and hsadmm_expand_dual under the union

Values follow the workloads of the repository: He-normal weights, replicas that differ from them by N(0, 1e-3),
duals N(0, 1e-4), global consensus N(0, 0.05^2), inter-node dual N(0, 0.01^2).
"""
import math

import torch

import paper_2512_14628_amd as hs

MODES = {"none": hs.MODE_NONE, "filter": hs.MODE_FILTER, "channel": hs.MODE_CHANNEL, "both": hs.MODE_BOTH}
FORMS = ("step", "predicted", "weighted", "norms", "retrain", "union")


# ------------------------------------------------------------------ cases

def listed():
    def case(name, form, net, blocks, width, mode, keep, R, spread=False):
        return {"name": name, "form": form, "net": net, "blocks": blocks, "width": width, "mode": mode, "keep": keep,
                "R": R, "spread": spread}

    return [
        # the smallest call: a tiny CNN of 5 layers, where launches and host work are all there is
        case("tiny_step", "step", "plain", "", 16, "filter", 0.5, 1),
        # a small network, one replica: ResNet-18
        case("resnet18_step", "step", "basic", "2-2-2-2", 64, "filter", 0.4, 1),
        # a network that has been shrunk before: odd widths, rows that are not whole 16-byte words, three replicas
        case("ragged_step", "step", "basic", "2-2-2-2", 45, "filter", 0.5, 3),
        # the benchmark's step: ResNet-50, four replicas, the first outer iterations
        case("resnet50_step", "step", "bottleneck", "3-4-6-3", 64, "filter", 0.4, 4),
        # ... once the pattern has settled and the previous selection is passed as a prediction
        case("resnet50_predicted", "predicted", "bottleneck", "3-4-6-3", 64, "filter", 0.4, 4),
        # ... with the inter-node terms and the residual norms: a whole dynamic outer iteration
        case("resnet50_norms", "norms", "bottleneck", "3-4-6-3", 64, "filter", 0.4, 4),
        # ... after the masks are frozen: what most of the iterations of a training run are
        case("resnet50_retrain", "retrain", "bottleneck", "3-4-6-3", 64, "filter", 0.4, 4),
        # ... the exchange under the union of two nodes' masks
        case("resnet50_union", "union", "bottleneck", "3-4-6-3", 64, "filter", 0.4, 4),
        # input-channel groups: ResNet-152, the plain and the full candidate
        case("resnet152_channel_step", "step", "bottleneck", "3-8-36-3", 64, "channel", 0.3, 4),
        case("resnet152_channel_weighted", "weighted", "bottleneck", "3-8-36-3", 64, "channel", 0.3, 4),
        # filter and channel constraints on every layer
        case("resnet50_both_step", "step", "bottleneck", "3-4-6-3", 64, "both", 0.6, 4),
        # the largest: every width times four, eight replicas, norms spread over four decades
        case("wide_step", "step", "bottleneck", "3-4-6-3", 256, "filter", 0.5, 8, True),
    ]


def draw(rng):
    """A network of any depth and width from a few tens of thousands of parameters to about 150 million (odd widths as
    often as even ones), any constraint, 1 to 8 replicas, any form of the step."""
    net = rng.choice(["plain", "basic", "basic", "bottleneck", "bottleneck", "bottleneck"])
    if net == "plain":
        blocks, top = "", 256
    elif net == "basic":
        blocks, top = "-".join(str(rng.randint(1, 3)) for _ in range(4)), 128
    else:
        blocks, top = "%d-%d-%d-%d" % (rng.randint(1, 3), rng.randint(1, 8), rng.randint(1, 24), rng.randint(1, 3)), 112
    width = int(round(12 * (top / 12) ** rng.random()))
    if rng.random() < 0.5:
        width -= width % 4                                   # whole 16-byte rows; the other half is as it falls
    return {"form": rng.choice(FORMS), "net": net, "blocks": blocks, "width": width,
            "mode": rng.choice(["filter", "filter", "channel", "both"]), "keep": round(rng.uniform(0.2, 0.8), 3),
            "R": rng.choice([1, 2, 3, 4, 4, 5, 6, 8]), "spread": rng.random() < 0.25}


# ------------------------------------------------------------------ networks

def _shapes(case):
    """(c_out, c_in, K_H*K_W) of every layer, the linear layer last."""
    w = case["width"]
    if case["net"] == "plain":
        return [(w, 3, 9), (2 * w, w, 9), (2 * w, 2 * w, 9), (4 * w, 2 * w, 9), (10, 4 * w, 1)]
    out, inp = [(w, 3, 49)], w
    for stage, count in enumerate(int(x) for x in case["blocks"].split("-")):
        ws = w << stage
        for b in range(count):
            if case["net"] == "basic":
                out += [(ws, inp, 9), (ws, ws, 9)]
                if b == 0 and inp != ws:
                    out.append((ws, inp, 1))
                inp = ws
            else:
                out += [(ws, inp, 1), (ws, ws, 9), (4 * ws, ws, 1)]
                if b == 0:
                    out.append((4 * ws, inp, 1))
                inp = 4 * ws
    return out + [(1000, inp, 1)]


def _kept(keep, groups):
    return max(1, min(groups, int(math.floor(keep * groups + 0.5))))


def _table(case):
    """The plan's layer table; the linear layer of the residual networks is left whole."""
    cols = {c: [] for c in ("elem_off", "c_out", "c_in", "khw", "mode", "k", "k_in")}
    off, shapes = 0, _shapes(case)
    for i, (co, ci, khw) in enumerate(shapes):
        off = (off + 3) // 4 * 4
        mode = "none" if i == len(shapes) - 1 and case["net"] != "plain" else case["mode"]
        keep = case["keep"]
        if case["spread"]:                                   # a keep ratio of every layer's own, around the case's
            keep = min(0.8, max(0.2, keep + 0.3 * math.sin(1 + 2.4 * i)))
        k = co if mode == "none" else _kept(keep, ci if mode == "channel" else co)
        for name, v in zip(cols, (off, co, ci, khw, MODES[mode], k, _kept(keep, ci) if mode == "both" else 0)):
            cols[name].append(v)
        off += co * ci * khw
    return cols, off


def _rows(cols):
    return [dict(zip(cols, vals)) for vals in zip(*cols.values())]


def _packed_elems(l, k, k_in):
    """Elements layer l packs when k groups (and, under both constraints, k_in channels) are kept."""
    if l["mode"] == hs.MODE_NONE:
        return l["c_out"] * l["c_in"] * l["khw"]
    if l["mode"] == hs.MODE_FILTER:
        return k * l["c_in"] * l["khw"]
    return (l["c_out"] if l["mode"] == hs.MODE_CHANNEL else k) * (k if l["mode"] == hs.MODE_CHANNEL else k_in) * l["khw"]


def _others(k, groups):
    """Groups the second node of the exchange keeps beside those the first one keeps."""
    return min(groups - k, k // 5)


# ------------------------------------------------------------------ one pass

def _inputs(case, seed):
    """The seed's tensors and the generator they were drawn from."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    cols, n = _table(case)
    layers, R, form = _rows(cols), case["R"], case["form"]

    def normal(sigma):
        return torch.randn(n, generator=gen, device=dev).mul_(sigma)

    base = torch.randn(n, generator=gen, device=dev)
    for l in layers:
        at = base[l["elem_off"]:l["elem_off"] + l["c_out"] * l["c_in"] * l["khw"]].view(l["c_out"], -1)
        at.mul_(math.sqrt(2.0 / (l["c_in"] * l["khw"])))
        if case["spread"]:
            at.mul_(torch.pow(10.0, torch.rand(l["c_out"], 1, generator=gen, device=dev) * 4 - 3))
    x = {"W": [normal(math.sqrt(1e-3)).add_(base) for _ in range(R)] if R > 1 else [base]}
    x["U"] = normal(1e-2)
    if form in ("weighted", "norms", "retrain", "union"):
        x["Zg"], x["Vd"] = normal(0.05), normal(0.01)
    if form == "norms":
        x["Zp"] = normal(0.05)
    return x, gen


def _other_mask(layers, mask, gen):
    """The mask of a second node that agrees with `mask` on all but a fifth of the groups."""
    other, at = mask.clone(), 0
    for l in layers:
        parts = {hs.MODE_NONE: [(l["c_out"], l["c_out"])], hs.MODE_FILTER: [(l["c_out"], l["k"])],
                 hs.MODE_CHANNEL: [(l["c_in"], l["k"])],
                 hs.MODE_BOTH: [(l["c_out"], l["k"]), (l["c_in"], l["k_in"])]}[l["mode"]]
        for groups, k in parts:
            more = _others(k, groups)
            if more:
                rank = torch.rand(groups, generator=gen, device=mask.device) + 2.0 * other[at:at + groups]
                other[at + torch.argsort(rank)[:more]] = 1
            at += groups
    return other


RHO1, RHO2, LAMBDA, NODES = 1.5e-3, 1.5e-4, 1e-4, 16         # penalties of Eq. (9), the same on every layer


def prepare(case, seed):
    x, gen = _inputs(case, seed)
    cols, n = _table(case)
    layers, R, form, dev = _rows(cols), case["R"], case["form"], x["U"].device
    s = {"form": form, "plan": hs.Plan(cols), **x}
    plan = s["plan"]
    s["Z"] = torch.zeros(n, device=dev)
    s["dst"] = torch.zeros(n, device=dev)
    s["mask"] = torch.zeros(plan.groups_total, dtype=torch.uint8, device=dev)
    s["packed"] = torch.zeros(plan.packed_capacity_elems, device=dev)
    s["off"] = torch.zeros(plan.n_layers + 1, dtype=torch.int64, device=dev)
    s["kept"] = torch.zeros(plan.groups_total, dtype=torch.int32, device=dev)
    s["ws"] = torch.zeros(plan.workspace_bytes, dtype=torch.uint8, device=dev)
    if form in ("weighted", "norms", "retrain", "union"):
        a, b = hs.hsadmm_node_coefficients([RHO1] * len(layers), [RHO2] * len(layers), LAMBDA, NODES, R)
        hs.hsadmm_plan_set_node_weights(plan, a, b)
        s["coef"] = torch.tensor([x for ab in zip(a, b) for x in ab], device=dev)
        s["norms"] = torch.zeros(4 * len(layers), dtype=torch.float64, device=dev)
    if form == "predicted":
        s["U_out"] = torch.zeros(n, device=dev)
        s["sel_prev"], s["sel"] = (torch.zeros(plan.groups_total, dtype=torch.int32, device=dev) for _ in range(2))
        hs.hsadmm_step(plan, s["W"], U=s["U"], U_out=s["U_out"], Z=s["Z"], mask=s["mask"], sel=s["sel_prev"],
                       workspace=s["ws"])
    elif form in ("retrain", "union"):
        # the masks the dynamic phase ended with, and the iteration that follows it
        hs.hsadmm_project_weighted(plan, s["W"], s["U"], s["Zg"], s["Vd"], s["Z"], None, s["mask"], None, s["ws"])
        if form == "retrain":
            hs.hsadmm_retrain_project(plan, s["W"], s["U"], s["Zg"], s["Vd"], s["Z"], None, s["mask"], False,
                                      s["packed"], s["off"], s["kept"], s["norms"], s["ws"])
        else:
            s["other"] = _other_mask(layers, s["mask"], gen)
            s["union"] = torch.zeros_like(s["other"])
    return s


def run(s):
    plan, form, ws = s["plan"], s["form"], s["ws"]
    if form == "step":
        hs.hsadmm_project_compact(plan, s["W"], s["U"], s["Z"], None, s["mask"], None, s["packed"], s["off"],
                                  s["kept"], ws)
        hs.hsadmm_expand(plan, s["packed"], None, s["dst"], ws)
        return [s[x] for x in ("U", "Z", "mask", "packed", "off", "kept", "dst")]
    if form == "predicted":
        hs.hsadmm_step(plan, s["W"], U=s["U"], U_out=s["U_out"], Z=s["Z"], mask=s["mask"], sel_prev=s["sel_prev"],
                       sel=s["sel"], packed=s["packed"], layer_off=s["off"], kept_idx=s["kept"], workspace=ws)
        hs.hsadmm_expand(plan, s["packed"], None, s["dst"], ws)
        return [s[x] for x in ("U_out", "Z", "mask", "sel", "packed", "off", "kept", "dst")]
    if form == "weighted":
        hs.hsadmm_project_weighted_compact(plan, s["W"], s["U"], s["Zg"], s["Vd"], s["Z"], None, s["mask"], None,
                                           s["packed"], s["off"], s["kept"], ws)
        hs.hsadmm_expand_dual(plan, s["packed"], None, s["dst"], s["Z"], s["Vd"], ws)
        return [s[x] for x in ("U", "Z", "mask", "packed", "off", "kept", "dst", "Vd")]
    if form == "norms":
        hs.hsadmm_step(plan, s["W"], U=s["U"], Zg=s["Zg"], Vd=s["Vd"], coef=s["coef"], Z=s["Z"], mask=s["mask"],
                       packed=s["packed"], layer_off=s["off"], kept_idx=s["kept"], residuals=s["norms"],
                       Zi_prev=s["Zp"], workspace=ws)
        hs.hsadmm_retrain_expand(plan, s["packed"], None, s["dst"], s["Z"], s["Vd"], s["Zg"], s["norms"], ws)
        return [s[x] for x in ("U", "Z", "mask", "packed", "off", "kept", "dst", "Vd", "norms")]
    if form == "retrain":
        hs.hsadmm_retrain_project(plan, s["W"], s["U"], s["Zg"], s["Vd"], s["Z"], None, s["mask"], True, s["packed"],
                                  s["off"], s["kept"], s["norms"], ws)
        hs.hsadmm_retrain_expand(plan, s["packed"], None, s["dst"], s["Z"], s["Vd"], s["Zg"], s["norms"], ws)
        return [s[x] for x in ("U", "Z", "packed", "off", "kept", "dst", "Vd", "norms")]
    hs.hsadmm_mask_or(plan, [s["mask"], s["other"]], s["union"])
    hs.hsadmm_compact_sum(plan, s["Z"], s["Vd"], s["union"], s["packed"], s["off"], s["kept"], ws)
    hs.hsadmm_expand_dual(plan, s["packed"], s["union"], s["dst"], s["Z"], s["Vd"], ws)
    return [s[x] for x in ("union", "packed", "off", "kept", "dst", "Vd")]


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Each input read once and each output written once, arena by arena (fp32)."""
    cols, _ = _table(case)
    layers, R, form = _rows(cols), case["R"], case["form"]
    n = sum(l["c_out"] * l["c_in"] * l["khw"] for l in layers)
    nk = sum(_packed_elems(l, l["k"], l["k_in"]) for l in layers)
    if form in ("step", "predicted"):
        # replicas and dual in, dual and Z out; packed out and in again; dst out
        return {"bytes": 4 * n * (R + 4) + 8 * nk, "flops": n * (R + 5)}
    if form == "weighted":
        # ... z and v in; the expansion reads Z and v and writes z and v
        return {"bytes": 4 * n * (R + 9) + 8 * nk, "flops": n * (R + 11)}
    if form == "norms":
        # ... the previous z_i and the previous z in
        return {"bytes": 4 * n * (R + 11) + 8 * nk, "flops": n * (3 * R + 20)}
    if form == "retrain":
        # as "norms", but z and v count on the kept groups only (a pruned group needs neither)
        return {"bytes": 4 * n * (R + 9) + 16 * nk, "flops": n * (3 * R + 15)}
    ku = sum(_packed_elems(l, l["k"] + _others(l["k"], l["c_in"] if l["mode"] == hs.MODE_CHANNEL else l["c_out"]),
                           l["k_in"] + _others(l["k_in"], l["c_in"])) for l in layers)
    # kept parts of Z and v in, packed out and in again; Z and v in, z and v out
    return {"bytes": 16 * n + 16 * ku, "flops": 2 * n + ku}


def tolerance(case):
    """fp32 values that are a few roundings deep, fp64 norms of them; masks, ranks and offsets are whole numbers and
    stay the same.  Against the same steps in fp64 the outputs are off by 3e-8 to 1.3e-7 in the 2-norm and by up to
    1e-5 in the worst element (a kept group's dual is what rounding leaves of it); four times that is allowed."""
    return {"rel": 5e-7, "max": 4e-5}


# ------------------------------------------------------------------ the same pass in 64 bits

def exact(case, seed):
    """What `run` returns for these inputs, from the definition of the step in plain torch, 64 bits throughout."""
    x, gen = _inputs(case, seed)
    cols, n = _table(case)
    layers, R, form = _rows(cols), case["R"], case["form"]
    mean = torch.zeros_like(x["U"], dtype=torch.float64)
    for w in x["W"]:
        mean += w
    mean /= R
    U = x["U"].double()
    dev = U.device
    a, b = 1.0, 0.0
    if "Zg" in x:
        gamma = LAMBDA / NODES + R * RHO1 + RHO2
        a, b = R * RHO1 / gamma, RHO2 / gamma
        z_old, v_old = x["Zg"].double(), x["Vd"].double()

    def part(t, l):
        return t[l["elem_off"]:l["elem_off"] + l["c_out"] * l["c_in"] * l["khw"]].view(l["c_out"], l["c_in"], l["khw"])

    def candidate(u):
        return mean + u if b == 0.0 else a * (mean + u) + b * (z_old - v_old)

    def largest(norms, k):
        m = torch.zeros(norms.numel(), dtype=torch.uint8, device=dev)
        m[torch.topk(norms, k).indices] = 1
        return m

    def selection(c):
        """Every layer's masks: [filters], [channels] or [filters, channels]."""
        masks = []
        for l in layers:
            sq = part(c, l).square().sum(2)
            if l["mode"] == hs.MODE_NONE:
                masks.append([torch.ones(l["c_out"], dtype=torch.uint8, device=dev)])
            elif l["mode"] == hs.MODE_CHANNEL:
                masks.append([largest(sq.sum(0), l["k"])])
            else:
                f = largest(sq.sum(1), l["k"])
                masks.append([f] if l["mode"] == hs.MODE_FILTER else [f, largest((sq * f[:, None]).sum(0), l["k_in"])])
        return masks

    def flat(masks):
        return torch.cat([m for ms in masks for m in ms])

    def sets(l, ms):
        """Indices of the layer's kept filters and channels."""
        f = torch.arange(l["c_out"], device=dev) if l["mode"] == hs.MODE_CHANNEL else ms[0].nonzero().flatten()
        ch = ms[-1].nonzero().flatten() if l["mode"] in (hs.MODE_CHANNEL, hs.MODE_BOTH) else torch.arange(l["c_in"], device=dev)
        return f, ch

    def keep(t, masks):
        out = torch.zeros_like(t)
        for l, ms in zip(layers, masks):
            f, ch = (i.view(s) for i, s in zip(sets(l, ms), ((-1, 1), (1, -1))))
            part(out, l)[f, ch] = part(t, l)[f, ch]
        return out

    def dual(u, z):
        out = u.clone()                                          # (the padding between layers is nobody's)
        for l in layers:
            part(out, l).copy_(part(u, l) + (part(mean, l) - part(z, l)))
        return out

    def shrink(t, masks):
        """packed, off and kept."""
        packed = torch.zeros(sum(l["c_out"] * l["c_in"] * l["khw"] for l in layers), dtype=torch.float64, device=dev)
        kept = torch.zeros(sum(m.numel() for ms in masks for m in ms), dtype=torch.int32, device=dev)
        off, at = [0], 0
        for l, ms in zip(layers, masks):
            f, ch = sets(l, ms)
            block = part(t, l)[f.view(-1, 1), ch.view(1, -1)].flatten()
            packed[off[-1]:off[-1] + block.numel()] = block
            off.append(off[-1] + block.numel())
            for m in ms:
                i = m.nonzero().flatten()
                kept[at:at + i.numel()] = i.int()
                at += i.numel()
        return packed, torch.tensor(off, dtype=torch.int64, device=dev), kept

    def ranks(masks):
        return torch.cat([torch.where(m > 0, m.int().cumsum(0).int() - 1, -1) for ms in masks for m in ms]).int()

    def sq(t, minus=None):
        return [float((part(t, l) - part(minus, l)).square().sum()) for l in layers]

    masks = selection(candidate(U))
    if form == "union":
        Z = keep(candidate(U), masks)
        other, at = _other_mask(layers, flat(masks), gen), 0
        both = []
        for ms in masks:
            row = []
            for m in ms:
                row.append(torch.maximum(m, other[at:at + m.numel()]))
                at += m.numel()
            both.append(row)
        z = keep(Z + v_old, both)
        return [flat(both), *shrink(Z + v_old, both), z, _on_layers(layers, v_old, Z - z)]
    z_before = x["Zp"].double() if form == "norms" else None
    if form == "retrain":                                        # two iterations before the one that is timed
        for _ in range(2):
            z_before = keep(candidate(U), masks)
            U = dual(U, z_before)
    Z = keep(candidate(U), masks)
    U = dual(U, Z)
    if form in ("step", "predicted"):
        head = [U, Z, flat(masks)] + ([ranks(masks)] if form == "predicted" else [])
        return head + [*shrink(Z, masks), Z]
    z = keep(Z + v_old, masks)
    out = [U, Z] + ([] if form == "retrain" else [flat(masks)]) + [*shrink(Z + v_old, masks), z,
                                                                   _on_layers(layers, v_old, Z - z)]
    if form == "weighted":
        return out
    primal = [sum(v) for v in zip(*(sq(w.double(), Z) for w in x["W"]))]
    return out + [torch.tensor(primal + sq(Z, z_before) + sq(Z, z) + sq(z, z_old), dtype=torch.float64, device=dev)]


def _on_layers(layers, t, d):
    """t + d where there are layers, t in the padding between them."""
    out = t.clone()
    for l in layers:
        at = slice(l["elem_off"], l["elem_off"] + l["c_out"] * l["c_in"] * l["khw"])
        out[at] += d[at]
    return out
