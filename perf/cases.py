"""Performance cases of the merged-gradient path: what a training job has this library do between the backward
pass and the next forward pass, over the range of models, worker counts, gradient types and call patterns it is
used with.

A case names a model (the tensors whose gradients are merged), the number of workers whose gradients the GPU
holds, the gradient type, the call pattern (`form`) and how the caller's tensors lie in memory (`views`: every
tensor a view into one dense flat buffer per role, as flattened parameters are, so that tensors start on any
element; otherwise every tensor has an allocation of its own).  Forms:

  fused      one group_pipeline call over all groups: everything is ready at once
  per_group  one group_pipeline call per group, as the communication handler sends them
  staged     pack, reduce and unpack_update over all groups: the exchange lies between them
  two_step   pack, then reduce_update, over all groups
  direct     direct_update over all groups: nothing has to be transmitted
  arrival    pack_tensors for every tensor as it arrives, reduce_update for a group once it is full
  local      one worker's share of a multi-GPU job: pack_tensors as tensors arrive, unpack_update at the end

`exact` restates the plan, the layout and the arithmetic in plain Python and torch, in 64 bits.
"""
import math

import numpy as np
import torch

import paper_1912_09268_amd as M

LR, MOMENTUM = 0.1, 0.9
BASE_GRANULE = 256                      # group bases are multiples of this many arena elements
DTYPES = {"f32": (torch.float32, 4, M.F32), "bf16": (torch.bfloat16, 2, M.BF16), "f16": (torch.float16, 2, M.F16)}


# ---- models: (elements, backward seconds) of every tensor in forward order, and (a, b) of the all-reduce ----------

def _timed(layers, seconds):
    """Backward times proportional to the work charged to each tensor."""
    total = sum(work for _, work in layers)
    return [n for n, _ in layers], [seconds * work / total for _, work in layers]


def _toy_mlp():
    sizes = [784 * 256, 256, 256 * 256, 256, 256 * 128, 128, 128 * 10, 10]
    return sizes, [5e-4 if n > 1000 else 5e-5 for n in sizes], 1e-5, 1e-9


def _resnet50():
    layers = []

    def conv_bn(cin, cout, k, hw):
        layers.append((cin * cout * k * k, 4 * cin * cout * k * k * hw * hw))
        layers.extend([(cout, 4 * cout * hw * hw)] * 2)

    conv_bn(3, 64, 7, 112)
    cin, hw = 64, 56
    for stage, (planes, blocks) in enumerate(((64, 3), (128, 4), (256, 6), (512, 3))):
        for block in range(blocks):
            out = hw // 2 if stage and not block else hw
            conv_bn(cin, planes, 1, hw)
            conv_bn(planes, planes, 3, out)
            conv_bn(planes, 4 * planes, 1, out)
            if not block:
                conv_bn(cin, 4 * planes, 1, out)
            cin, hw = 4 * planes, out
    layers += [(2048 * 1000, 4 * 2048 * 1000), (1000, 1000)]
    return (*_timed(layers, 0.1), 2e-5, 1e-10)


def _vgg16():
    layers = []
    for cin, cout, hw in ((3, 64, 224), (64, 64, 224), (64, 128, 112), (128, 128, 112), (128, 256, 56), (256, 256, 56),
                          (256, 256, 56), (256, 512, 28), (512, 512, 28), (512, 512, 28), (512, 512, 14),
                          (512, 512, 14), (512, 512, 14)):
        layers += [(9 * cin * cout, 36 * cin * cout * hw * hw), (cout, cout * hw * hw)]
    for fin, fout in ((25088, 4096), (4096, 4096), (4096, 1000)):
        layers += [(fin * fout, 4 * fin * fout), (fout, fout)]
    return (*_timed(layers, 0.19), 2e-5, 8e-11)


def _transformer():
    h, f, vocab, seq, tokens = 1024, 4096, 30522, 512, 4096
    linear = lambda i, o: [(i * o, 4 * i * o * tokens), (o, o * tokens)]  # noqa: E731
    norm = [(h, 4 * h * tokens)] * 2
    layers = [(vocab * h, h * tokens), (seq * h, h * tokens), (2 * h, h * tokens)] + norm
    for _ in range(24):
        for _ in range(4):
            layers += linear(h, h)
        layers += norm + linear(h, f) + linear(f, h) + norm
    layers += linear(h, h)
    return (*_timed(layers, 0.51), 1e-5, 4e-11)


def _many(case):
    """Tensor sizes around a median, log-normal: the many-small-layers models."""
    rng = np.random.default_rng(case["sizes_seed"])
    raw = np.exp(rng.normal(math.log(case["median"]), case["spread"], case["L"]))
    sizes = np.clip(np.rint(raw), 1, 64 * case["median"]).astype(np.int64)
    return [int(x) for x in sizes], [float(x) for x in rng.uniform(2e-5, 2e-4, case["L"])], 5e-5, 2e-10


def _model(case):
    named = {"toy_mlp": _toy_mlp, "resnet50": _resnet50, "vgg16": _vgg16, "transformer": _transformer}
    return named[case["model"]]() if case["model"] in named else _many(case)


# ---- cases --------------------------------------------------------------------------------------------------------

def _case(name, model, P, dtype, form, views=False, **more):
    return dict(name=name, model=model, P=P, dtype=dtype, form=form, views=views, **more)


TINY = dict(L=1000, median=4096, spread=1.5, sizes_seed=191209268)


def listed():
    return [
        # a small multi-layer perceptron on 4 workers: the smallest call, all latency
        _case("mlp fused", "toy_mlp", 4, "f32", "fused"),
        # the same through the handler: a launch for each of its few small groups
        _case("mlp per group", "toy_mlp", 4, "f32", "per_group"),
        # ResNet-50 on 8 workers, everything ready at once
        _case("resnet50 fused", "resnet50", 8, "f32", "fused"),
        # ResNet-50 the way the handler sends it during the backward pass
        _case("resnet50 per group", "resnet50", 8, "f32", "per_group"),
        # half-precision ResNet-50 gradients with an exchange between the steps, 4 workers
        _case("resnet50 f16 staged", "resnet50", 4, "f16", "staged"),
        # one GPU's share of a real multi-GPU job: gradients packed as they arrive, update at the end
        _case("resnet50 local", "resnet50", 1, "f32", "local"),
        # 32 workers' half-size gradients, flattened parameters
        _case("resnet50 bf16 32 workers", "resnet50", 32, "bf16", "two_step", views=True),
        # VGG-16, one tensor of which holds three quarters of the model: the headline and the largest call
        _case("vgg16 fused", "vgg16", 8, "f32", "fused"),
        # mixed-precision transformer
        _case("transformer bf16 fused", "transformer", 8, "bf16", "fused"),
        # the same on a worker count that is no power of two, nothing transmitted
        _case("transformer bf16 direct", "transformer", 6, "bf16", "direct"),
        # a thousand small layers of ragged sizes, 16 workers
        _case("tiny layers fused", "many", 16, "f32", "fused", **TINY),
        # a thousand small layers as flat-buffer views, packed as they arrive, 3 workers
        _case("tiny layers arrival", "many", 3, "f32", "arrival", views=True, **TINY),
    ]


def draw(rng):
    dtype = rng.choice(["f32", "f32", "bf16", "f16"])
    form = rng.choice(["fused", "fused", "per_group", "staged", "two_step", "direct", "arrival", "local"])
    P = 1 if form == "local" else rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16, 24, 32])
    L = int(round(math.exp(rng.uniform(math.log(6), math.log(1000)))))
    largest = min(8e5, 1.2e8 / L / P)          # keeps the bytes of a pass well below the largest listed case's
    median = int(round(math.exp(rng.uniform(math.log(200), math.log(max(400, largest))))))
    return dict(model="many", P=P, dtype=dtype, form=form, views=rng.random() < 0.4, L=L, median=median,
                spread=round(rng.uniform(0.3, 1.8), 3), sizes_seed=rng.randrange(1 << 30))


# ---- inputs -------------------------------------------------------------------------------------------------------

class Slab:
    """Tensors of one role.  Dense views, or each at the alignment an allocation of its own would have."""

    def __init__(self, sizes, dtype, views):
        item = torch.empty(0, dtype=dtype).element_size()
        self.sizes, self.at, end = sizes, [], 0
        for n in sizes:
            align = 1 if views else max(1, (2 << 20 if n * item > 1 << 20 else 512) // item)
            end = -(-end // align) * align
            self.at.append(end)
            end += n
        self.flat = torch.zeros(max(end, 1), dtype=dtype, device="cuda")

    def pointers(self):
        item = self.flat.element_size()
        return [self.flat.data_ptr() + item * at for at in self.at]

    def parts(self):
        return [self.flat[at:at + n] for at, n in zip(self.at, self.sizes)]


def _inputs(case, seed):
    sizes = _model(case)[0]
    dtype = DTYPES[case["dtype"]][0]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    grads = [Slab(sizes, dtype, case["views"]) for _ in range(case["P"])]
    for g in grads:
        g.flat.normal_(0.0, 1e-2, generator=gen)
    w, v = (Slab(sizes, torch.float32, case["views"]) for _ in range(2))
    w.flat.normal_(0.0, 1.0, generator=gen)
    v.flat.normal_(0.0, 1e-2, generator=gen)
    return grads, w, v, gen


def _table(pointers):
    return torch.tensor(pointers, dtype=torch.int64).cuda()


def prepare(case, seed):
    sizes, t_b, a, b = _model(case)
    dtype, item, code = DTYPES[case["dtype"]]
    merged, _ = M.plan([n * item for n in sizes], t_b, a, b)
    ctx = M.Context(sizes, merged, case["P"], code)
    grads, w, v, gen = _inputs(case, seed)
    merge = Slab([ctx.arena_elems] * case["P"], dtype, False)
    reduced = torch.zeros(ctx.arena_elems, dtype=torch.float32, device="cuda")
    if case["form"] == "local":                                       # what the exchange would have delivered
        reduced.normal_(0.0, 1e-2, generator=gen)
    state = dict(case=case, ctx=ctx, merged=[int(x) for x in merged], keep=grads, w=w.flat, v=v.flat,
                 merge=merge.flat, reduced=reduced,
                 g_ptrs=_table([p for g in grads for p in g.pointers()]), m_ptrs=_table(merge.pointers()),
                 w_ptrs=_table(w.pointers()), v_ptrs=_table(v.pointers()))
    state["args"] = {k: state[k].data_ptr() for k in ("g_ptrs", "m_ptrs", "w_ptrs", "v_ptrs", "reduced")}
    return state


def run(state):
    ctx, form, p = state["ctx"], state["case"]["form"], state["args"]
    stream = torch.cuda.current_stream().cuda_stream
    g, m, r, w, v = p["g_ptrs"], p["m_ptrs"], p["reduced"], p["w_ptrs"], p["v_ptrs"]
    out = {"w": state["w"], "v": state["v"]}
    if form == "fused":
        ctx.group_pipeline(-1, g, m, r, w, v, LR, MOMENTUM, stream)
        out.update(merge=state["merge"], reduced=state["reduced"])
    elif form == "per_group":
        for k in range(ctx.n_groups):
            ctx.group_pipeline(k, g, m, r, w, v, LR, MOMENTUM, stream)
        out.update(merge=state["merge"], reduced=state["reduced"])
    elif form == "staged":
        ctx.pack(-1, g, m, stream)
        ctx.reduce(-1, m, r, stream)
        ctx.unpack_update(-1, r, w, v, LR, MOMENTUM, stream)
        out.update(merge=state["merge"], reduced=state["reduced"])
    elif form == "two_step":
        ctx.pack(-1, g, m, stream)
        ctx.reduce_update(-1, m, w, v, LR, MOMENTUM, stream)
        out.update(merge=state["merge"])
    elif form == "direct":
        ctx.direct_update(-1, g, 0, w, v, LR, MOMENTUM, stream)
    elif form == "arrival":
        k = 0
        for i in range(ctx.L - 1, -1, -1):
            ctx.pack_tensors(i, i, g, m, stream)
            if not state["merged"][i]:
                ctx.reduce_update(k, m, w, v, LR, MOMENTUM, stream)
                k += 1
        out.update(merge=state["merge"])
    else:
        for i in range(ctx.L - 1, -1, -1):
            ctx.pack_tensors(i, i, g, m, stream)
        ctx.unpack_update(-1, r, w, v, LR, MOMENTUM, stream)
        out.update(merge=state["merge"])
    return out


# ---- what a pass cannot do without, and what it has to give -------------------------------------------------------

def work(case):
    n, P, g = sum(_model(case)[0]), case["P"], DTYPES[case["dtype"]][1]
    pack, summed, update = 2 * P * g, P, 4               # bytes, additions and products per element
    each = {"fused": (pack + 20, summed + update), "per_group": (pack + 20, summed + update),
            "staged": (pack + (P * g + 4) + 20, summed + update), "two_step": (pack + P * g + 16, summed + update),
            "direct": (P * g + 16, summed + update), "arrival": (pack + P * g + 16, summed + update),
            "local": (pack + 20, update)}[case["form"]]
    return {"bytes": n * each[0], "flops": n * each[1]}


def tolerance(case):
    """The arithmetic is promised operation by operation (binary32, sums in worker order, one rounding each), so
    every implementation of it gives the same bits."""
    return "exact"


def _groups(sizes_bytes, t_b, a, b):
    """Algorithm 1: tensors from the last to the first; one is merged into the next if that one's gradient exists
    less than `a` after its own message could start."""
    L, ready, now = len(t_b), [0.0] * len(t_b), 0.0
    for i in range(L - 1, -1, -1):
        now += t_b[i]
        ready[i] = now
    groups, start, size = [[L - 1]], ready[L - 1], sizes_bytes[L - 1]
    for i in range(L - 2, -1, -1):
        if ready[i] - start < a:
            groups[-1].append(i)
            start, size = max(start, ready[i]), size + sizes_bytes[i]
        else:
            groups.append([i])
            start, size = max(start + (a + b * size), ready[i]), sizes_bytes[i]
    return groups


def exact(case, seed):
    sizes, t_b, a, b = _model(case)
    dtype, item, _ = DTYPES[case["dtype"]]
    form, P = case["form"], case["P"]
    place, end = [0] * len(sizes), 0                     # where each tensor lies in an arena
    for members in _groups([n * item for n in sizes], t_b, a, b):
        end = -(-end // BASE_GRANULE) * BASE_GRANULE
        for i in members:
            place[i] = end
            end += sizes[i]
    arena = -(-end // BASE_GRANULE) * BASE_GRANULE
    grads, w, v, gen = _inputs(case, seed)
    out = {}
    if form != "direct":
        merge = Slab([arena] * P, dtype, False)
        for m, g in zip(merge.parts(), grads):
            for i, part in enumerate(g.parts()):
                m[place[i]:place[i] + sizes[i]] = part
        out["merge"] = merge.flat
    if form == "local":
        given = torch.zeros(arena, dtype=torch.float32, device="cuda").normal_(0.0, 1e-2, generator=gen)
        mean = [given[place[i]:place[i] + n].double() for i, n in enumerate(sizes)]
    else:
        total = grads[0].flat.double()
        for g in grads[1:]:
            total += g.flat
        total *= 1.0 / P
        mean = [total[at:at + n] for at, n in zip(grads[0].at, sizes)]
    if form in ("fused", "per_group", "staged"):
        out["reduced"] = torch.zeros(arena, dtype=torch.float64, device="cuda")
        for i, n in enumerate(sizes):
            out["reduced"][place[i]:place[i] + n] = mean[i]
    out["w"], out["v"] = w.flat.double(), v.flat.double()
    lr, mu = float(np.float32(LR)), float(np.float32(MOMENTUM))
    for at, n, r in zip(w.at, sizes, mean):
        step = out["v"][at:at + n].mul_(mu).add_(r)
        out["w"][at:at + n].sub_(step, alpha=lr)
    return out
