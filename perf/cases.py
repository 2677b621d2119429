"""The work whose time matters: whole rounds of resident tenants, as a serving process runs them.

A case names the tenants that share the GPU (family:batch:extent, the extent being the image side or the token count), their
element type, how a round is issued, and the regulation plan.  `prepare` does what such a process does once -- weights and
activations resident in device memory, a context, streams, a plan -- and `run` is one round through the session's `run`,
which returns when every tenant has produced its output.
"""
import functools
import math

import torch

from paper_2304_11745_amd import binding as B
from paper_2304_11745_amd import harness
from synth import graphs as G

MODES = {"sequential": B.GACER_MODE_SEQUENTIAL, "parallel": B.GACER_MODE_STREAM_PARALLEL, "regulated": B.GACER_MODE_PLAN}

FAMILIES = {
    "toy_cnn": lambda dt, n, ext: G.toy_cnn(dt, n, ext),
    "toy_mlp": lambda dt, n, ext: G.toy_mlp(dt, n),
    "alexnet": lambda dt, n, ext: G.alexnet(dt, n, ext),
    "vgg16": lambda dt, n, ext: G.vgg16(dt, n, ext),
    "resnet18": lambda dt, n, ext: G.resnet18(dt, n, ext),
    "resnet34": lambda dt, n, ext: G.resnet34(dt, n, ext),
    "resnet50": lambda dt, n, ext: G.resnet50(dt, n, ext),
    "resnet101": lambda dt, n, ext: G.resnet101(dt, n, ext),
    "densenet121": lambda dt, n, ext: G.densenet121(dt, n, ext),
    "mobilenetv2": lambda dt, n, ext: G.mobilenetv2(dt, n, ext),
    "mobilenetv3": lambda dt, n, ext: G.mobilenetv3_large(dt, n, ext),
    "bert": lambda dt, n, ext: G.bert_base(dt, n, ext),
}


def listed():
    return [
        # the smallest deployment: two toy tenants, six launches; the round is launch and synchronisation latency
        dict(name="toy_pair", tenants="toy_cnn:1:32,toy_mlp:4:1", dtype="f32", mode="parallel", threads=False, plan=""),
        # one image through one mobile network: a chain of fifty dependent kernels of a few microseconds
        dict(name="one_image", tenants="mobilenetv2:1:224", dtype="bf16", mode="sequential", threads=False, plan=""),
        # a short request to a text encoder, a token count that is no multiple of a tile
        dict(name="text_request", tenants="bert:2:72", dtype="bf16", mode="sequential", threads=False, plan=""),
        # eight batch-1 tenants, one issuing thread each: the multi-tenant serving case that is bound by launches
        dict(name="eight_batch1", tenants="resnet18:1:224,resnet18:1:224,resnet50:1:224,resnet50:1:224,mobilenetv2:1:224,"
             "mobilenetv2:1:224,vgg16:1:224,vgg16:1:224", dtype="bf16", mode="parallel", threads=True, plan=""),
        # the benchmark's headline workload
        dict(name="headline_f32", tenants="resnet18:8:224,mobilenetv2:8:224", dtype="f32", mode="parallel", threads=False, plan=""),
        # three image tenants at throughput batch sizes, in bf16
        dict(name="images_bf16", tenants="resnet50:16:224,vgg16:8:224,mobilenetv2:32:224", dtype="bf16", mode="parallel", threads=False, plan=""),
        # the same kind of mix under a regulation plan: decomposed operators and pointers
        dict(name="regulated_bf16", tenants="resnet50:16:224,vgg16:8:224,mobilenetv3:32:224", dtype="bf16", mode="regulated",
             threads=False, plan="batch2@1,cout2@0,pointers1"),
        # text and image tenants together, the widest mix
        dict(name="text_and_images", tenants="bert:8:128,resnet50:32:224,vgg16:16:224,mobilenetv2:64:224", dtype="bf16",
             mode="parallel", threads=False, plan=""),
        # fp32 convolution throughput: one large tenant beside two small ones
        dict(name="mix_f32", tenants="alexnet:8:224,vgg16:8:224,resnet18:8:224", dtype="f32", mode="parallel", threads=False, plan=""),
        # deep tenants: more than three hundred short launches a round
        dict(name="deep_bf16", tenants="resnet101:8:224,densenet121:8:224,mobilenetv3:8:224", dtype="bf16", mode="parallel",
             threads=True, plan=""),
        # odd batches and image extents, fp32, decomposed along the output channels
        dict(name="ragged_f32", tenants="resnet34:3:193,densenet121:5:161,mobilenetv3:7:147", dtype="f32", mode="regulated",
             threads=False, plan="cout2@0"),
        # large batches, one tenant after another: what the convolution kernels reach when nothing runs beside them
        dict(name="large_batch", tenants="vgg16:32:224,resnet18:32:224", dtype="bf16", mode="sequential", threads=False, plan=""),
    ]


def draw(rng):
    while True:
        if rng.random() < 0.1:
            case = dict(tenants="toy_cnn:%d:%d,toy_mlp:%d:1" % (_log(rng, 1, 64), _log(rng, 9, 128), _log(rng, 1, 512)))
        else:
            names = [n for n in FAMILIES if not n.startswith("toy")]
            parts = []
            for name in (rng.choice(names) for _ in range(rng.choice([1, 1, 2, 2, 3, 3, 4, 6]))):
                ext = 8 * rng.randint(2, 32) if name == "bert" else _log(rng, 96, 256) if rng.random() < 0.5 else 224
                parts.append("%s:%d:%d" % (name, _log(rng, 1, 64), ext))
            case = dict(tenants=",".join(parts))
        case.update(dtype=rng.choice(["f32", "bf16"]), mode=rng.choice(list(MODES)), threads=rng.random() < 0.4, plan="")
        if case["mode"] == "regulated":
            case["plan"] = rng.choice(["batch2@0", "cout2@0", "batch4@0,pointers1", "cout2@0,pointers2", "pointers1"])
        if _cost(case) <= _largest():
            return case


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


@functools.lru_cache(maxsize=1)
def _largest():
    return max(_cost(c) for c in listed())


def _cost(case):
    """Rough seconds of a pass, for comparing cases: matrix work, memory traffic and one launch per operator."""
    w = work(case)
    launches = sum(len(t.ops) for t in _tenants(case))
    return w["flops"] / (4e14 if case["dtype"] == "bf16" else 1e14) + w["bytes"] / 3e12 + launches * 4e-6


def _tenants(case):
    out = []
    for part in case["tenants"].split(","):
        name, batch, ext = part.split(":")
        out.append(FAMILIES[name](case["dtype"], int(batch), int(ext)))
    return out


def _draw_tenant(tenant, seed):
    """Input and parameters of a tenant as host arrays in logical order: uniform images or N(0, 0.02^2) token rows, He-uniform
    weights with the folded normalisation, small biases and shifts."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def uniform(shape, bound):
        return torch.rand(shape, generator=gen, device="cuda").mul_(2 * bound).sub_(bound)
    shape = tenant.tensors[tenant.input]
    if tenant.input_dist == "normal002":
        x = torch.randn(shape, generator=gen, device="cuda").mul_(0.02)
    else:
        x = uniform(shape, 1.0)
    params = []
    for p in tenant.params:
        if p.init == "he_uniform":
            a = uniform(p.shape, math.sqrt(6.0 / p.fan_in) * p.fold)
        elif p.init == "ones":
            a = uniform(p.shape, 0.05).add_(1.0).mul_(p.fold)
        elif p.init == "zeros":
            a = uniform(p.shape, 0.02)
        else:
            a = uniform(p.shape, p.fold)
        params.append(a.cpu().numpy())
    return x.cpu().numpy(), params


def _plan(sess, text):
    """`axisF@T` decomposes every operator of tenant T that allows it F ways along the axis; `pointersP` cuts every tenant into
    P + 1 segments of equal length."""
    splits, edges = [], []
    for item in text.split(","):
        if item.startswith("pointers"):
            k = int(item[len("pointers"):])
            edges = sess.edges_from_pointers([[len(t.ops) * (j + 1) // (k + 1) for j in range(k)] for t in sess.tenants])
        else:
            what, tenant = item.split("@")
            splits += sess.uniform_splits(what[:-1], int(what[-1]), tenants=[int(tenant)])
    sess.set_plan(splits, edges)


def prepare(case, seed):
    tenants = _tenants(case)
    sess = harness.Session(tenants, [_draw_tenant(t, seed * 64 + i) for i, t in enumerate(tenants)])
    if case["threads"]:
        sess.set_issue_threads(True)
    if case["plan"]:
        _plan(sess, case["plan"])
    return dict(session=sess, mode=MODES[case["mode"]], outputs=[sess.acts[i][t.output] for i, t in enumerate(tenants)])


def run(state):
    state["session"].run(state["mode"], 1)
    return state["outputs"]


def work(case):
    """Every parameter and every tenant's input read once, every operator's output tensor (which the caller owns) written
    once; two operations per multiply-accumulate."""
    esz = 2 if case["dtype"] == "bf16" else 4
    flops = nbytes = 0
    for t in _tenants(case):
        flops += 2 * G.gemm_macs(t)
        weights = {op.w for op in t.ops}
        nbytes += esz * math.prod(t.tensors[t.input])
        nbytes += sum((esz if i in weights else 4) * math.prod(p.shape) for i, p in enumerate(t.params))
        nbytes += sum(esz * math.prod(t.tensors[op.out]) for op in t.ops)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the difference measured against the same networks evaluated with 64-bit sums (every tensor stored in
    the tenant's type on both sides): fp32 at most 1.8e-6, bf16 at most 7.8e-3, deep networks compounding their roundings."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 3e-2, "max": 3e-1}
