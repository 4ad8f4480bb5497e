"""What the performance of this library is measured on.

A case is a set of member models fused into one DAG, a batch, an image side and the way the DAG is used:

* "run":   a resident handle, one shared input batch, one pass of the launch schedule (fi_run);
* "serve": a resident handle whose members bring inputs and batches of their own (fi_run_batches, the call the
           request aggregator makes once per round); member i brings `batch`, less 3 i, but at least one image;
* "swap":  a request that meets a cold device: build the DAG from packed models in pinned memory, load it, run one
           batch, unload it.

Weights are He-normal with N(0, 0.1) biases and images N(0, 1), the distributions of this repository's benchmark and
tests (the fp32 pair of tiny networks: zero biases, U[0, 1) images), drawn on the GPU from the seed.  Members named in WIDE
keep fp32-stored activations, as in the benchmark: with such weights they amplify bf16 storage rounding beyond the parity
bar.  Outputs are every member's logits (or probabilities) for every image.
"""
import math

import torch

import paper_2410_21120_amd as fi
from workloads import gen, zoo

WIDE = {"mobilenetv2", "mobilenet_v3_large"}
# Relative L2 between two executors that round storage at the same places and sum in different precision (the CPU
# oracle's fp32 and fp64 builds; two weight seeds, one image): 0.0004 (SqueezeNet) to 0.0036 for most families with bf16
# storage, 0.0044 to 0.0064 for these; 1.5e-6 to 5e-6 for fp32-stored activations, whose inputs are split into two bf16 terms
# (16 mantissa bits: the representation itself is good for 1e-4 on these networks); 2e-7 to 2.3e-6 for fp32 models.  The largest
# single difference, over the value or the result's root mean square, is three to four times the relative L2.
ROUGH = {"vgg11", "vgg16", "mobilenet_v3_small", "mnasnet1_0", "shufflenet_v2_x1_0"}


def listed():
    return [
        # the smallest calls: two tiny fp32 networks, one 32 x 32 image; latency only
        dict(name="tiny_fp32_x2_b1", mode="run", members="tiny*2", dtype="f32", batch=1, side=32, chunks=0),
        # interactive inference: two small members, one image
        dict(name="resnet18_x2_b1", mode="run", members="resnet18*2", dtype="bf16", batch=1, side=224, chunks=0),
        # an unconverted fp32 model at a small batch
        dict(name="resnet18_fp32_b4", mode="run", members="resnet18", dtype="f32", batch=4, side=224, chunks=0),
        # a heterogeneous DAG: dense, depthwise and fully connected layers side by side, a medium batch
        dict(name="mixed3_b8", mode="run", members="resnet50+mobilenetv2+vgg16", dtype="bf16", batch=8, side=224, chunks=0),
        # a serving round: four resident models, ragged batches 7, 4, 1, 1 of their own images
        dict(name="serve4_b7", mode="serve", members="resnet18+resnet50+mobilenetv2+vgg16", dtype="bf16", batch=7, side=224, chunks=0),
        # a swap request on a cold device: build, load, run, unload
        dict(name="swap4_b8", mode="swap", members="resnet18+resnet50+mobilenetv2+vgg16", dtype="bf16", batch=8, side=224, chunks=0),
        # an odd batch of odd-sized images through branching modules with concatenations
        dict(name="googlenet_x3_b13", mode="run", members="googlenet*3", dtype="bf16", batch=13, side=203, chunks=0),
        # a mobile family with fp32-stored activations: depthwise layers, squeeze-excite gates
        dict(name="mobilenetv3_x4_b32", mode="run", members="mobilenet_v3_large*4", dtype="bf16", batch=32, side=224, chunks=0),
        # many narrow layers and concatenations
        dict(name="densenet121_x4_b32", mode="run", members="densenet121*4", dtype="bf16", batch=32, side=224, chunks=0),
        # grouped convolutions
        dict(name="resnext101_x4_b32", mode="run", members="resnext101_32x8d*4", dtype="bf16", batch=32, side=224, chunks=0),
        # one large model, a large batch: throughput of a single member
        dict(name="vgg16_b64", mode="run", members="vgg16", dtype="bf16", batch=64, side=224, chunks=0),
        # the benchmark's headline: eight members, the early levels in two member chunks
        dict(name="resnet50_x8_b32", mode="run", members="resnet50*8", dtype="bf16", batch=32, side=224, chunks=2),
    ]


def families(case):
    names = []
    for part in case["members"].split("+"):
        fam, _, count = part.partition("*")
        names += [fam] * int(count or 1)
    return names


def model_of(case, fam):
    return zoo.tiny_cnn("f32") if fam == "tiny" else zoo.FAMILIES[fam](dtype=case["dtype"], hw=case["side"])


def batches(case):
    n = len(families(case))
    return [max(1, case["batch"] - 3 * i) for i in range(n)] if case["mode"] == "serve" else [case["batch"]] * n


def multiply_adds(case):
    one = {fam: model_of(case, fam).macs() for fam in set(families(case))}
    return sum(one[fam] * b for fam, b in zip(families(case), batches(case)))


MOST_BF16, MOST_F32 = 0.4e12, 7.2e9   # multiply-adds of a drawn case: below the largest listed case of the data type


def draw(rng):
    def spread(lo, hi):   # over the logarithm, odd values among them
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    dense = ["resnet18", "resnet34", "resnet50", "resnet101", "wide_resnet50_2", "resnext50_32x4d", "alexnet", "vgg11", "vgg16",
             "squeezenet1_1", "googlenet", "densenet121", "mobilenetv2", "mobilenet_v3_large", "mobilenet_v3_small", "mnasnet1_0",
             "shufflenet_v2_x1_0", "inception_v3"]
    while True:
        mode = rng.choice(["run", "run", "run", "run", "serve", "swap"])
        side, chunks, dtype = rng.randint(97, 256), 0, "bf16"
        if mode == "run" and rng.random() < 0.2:
            dtype = "f32"
            fam = rng.choice(["tiny", "resnet18", "squeezenet1_1", "mobilenetv2"])
            members, batch = "%s*%d" % (fam, spread(1, 4)), spread(1, 8)
            side = 32 if fam == "tiny" else side
        elif mode == "run":
            kinds = rng.sample(dense, rng.choice([1, 1, 2, 3]))
            counts = [spread(1, 8) if len(kinds) == 1 else rng.randint(1, 2) for _ in kinds]
            members, batch = "+".join("%s*%d" % kc for kc in zip(kinds, counts)), spread(1, 64)
            chunks = rng.choice([0, 0, 2]) if counts[0] >= 4 else 0
        else:
            members = "+".join(rng.sample(["resnet18", "resnet50", "mobilenetv2", "vgg16"], rng.randint(2, 4)))
            batch = rng.randint(1, 8)
        case = dict(mode=mode, members=members, dtype=dtype, batch=batch, side=side, chunks=chunks)
        if len(families(case)) * batch <= 128 and multiply_adds(case) <= (MOST_F32 if dtype == "f32" else MOST_BF16):
            return case


def weights(model, seed, zero_bias):
    """The model's canonical blob: He-normal weights and normal biases, drawn on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    blob = torch.zeros(gen.layout_blob(model), dtype=torch.uint8, device="cuda")
    stored, size = (torch.float32, 4) if model.dtype == "f32" else (torch.bfloat16, 2)
    for layer in model.layers:
        taps = layer.k * (layer.kw or layer.k)
        fan_in = {zoo.CONV: layer.cin // layer.groups * taps, zoo.DWCONV: taps, zoo.FC: layer.cin}.get(layer.op)
        if fan_in is None:
            continue
        n = layer.cout * fan_in
        blob[layer.w_off:layer.w_off + n * size].view(stored).copy_(torch.randn(n, generator=g, device="cuda") * math.sqrt(2.0 / fan_in))
        if layer.bias and not zero_bias:
            blob[layer.b_off:layer.b_off + 4 * layer.cout].view(torch.float32).copy_(torch.randn(layer.cout, generator=g, device="cuda") * 0.1)
    return blob.cpu()


def prepare(case, seed):
    fams, mode = families(case), case["mode"]
    models = [model_of(case, fam) for fam in fams]
    g = torch.Generator(device="cuda").manual_seed(seed)
    stored = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    tiny = fams[0] == "tiny"
    own = batches(case)

    def image_batch(b):
        shape = (b, case["side"], case["side"], 3)
        x = torch.rand(shape, generator=g, device="cuda") if tiny else torch.randn(shape, generator=g, device="cuda")
        return x.to(stored).contiguous()

    inputs = [image_batch(b) for b in own] if mode == "serve" else [image_batch(case["batch"])]
    outputs = [torch.zeros((b, m.layers[-1].cout), dtype=torch.float32, device="cuda") for m, b in zip(models, own)]
    specs, keep = [], []
    for i, (fam, model) in enumerate(zip(fams, models)):
        blob = weights(model, seed * 64 + i + 1, tiny)
        act = "f32" if fam in WIDE and case["dtype"] == "bf16" else None
        spec, alive = fi.make_spec(model, blob.data_ptr(), blob.numel(), act_dtype=act)
        if mode == "swap":   # the repository of models holds them in device layout, in pinned memory
            size = fi.fi_model_packed_size(spec)
            packed = torch.empty(size, dtype=torch.uint8, pin_memory=True)
            fi.fi_model_pack(spec, packed.data_ptr(), size)
            blob = packed
            spec, alive = fi.make_spec(model, blob.data_ptr(), size, act_dtype=act, packed=True)
        specs.append(spec)
        keep.append((blob, alive))
    state = dict(mode=mode, batch=case["batch"], own=own, inputs=inputs, outputs=outputs, in_ptrs=[x.data_ptr() for x in inputs],
                 out_ptrs=[y.data_ptr() for y in outputs], stream=torch.cuda.current_stream().cuda_stream, specs=specs, keep=keep,
                 allocators=fi.TorchAllocators("cuda:0"))
    if mode != "swap":
        state["dag"] = fi.Dag(specs, max(own), state["allocators"], keepalive=keep, per_member_inputs=mode == "serve",
                              member_chunks=case["chunks"])
        state["dag"].load(state["stream"])
    return state


def run(state):
    if state["mode"] == "run":
        state["dag"].run(state["in_ptrs"][0], state["batch"], state["out_ptrs"], state["stream"])
    elif state["mode"] == "serve":
        state["dag"].run_batches(state["in_ptrs"], state["own"], state["out_ptrs"], state["stream"])
    else:
        dag = fi.Dag(state["specs"], state["batch"], state["allocators"], keepalive=state["keep"], load_mode=fi.FI_LOAD_AUTO)
        dag.load(state["stream"])
        dag.run(state["in_ptrs"][0], state["batch"], state["out_ptrs"], state["stream"])
        dag.unload()
        dag.destroy()
    return state["outputs"]


def exact(case, seed):
    """Every member's outputs with its layers written out in plain torch, all values in 64 bits (nothing is rounded in storage)."""
    fams = families(case)
    models = [model_of(case, fam) for fam in fams]
    g = torch.Generator(device="cuda").manual_seed(seed)
    stored = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    tiny = fams[0] == "tiny"

    def image_batch(b):
        shape = (b, case["side"], case["side"], 3)
        x = torch.rand(shape, generator=g, device="cuda") if tiny else torch.randn(shape, generator=g, device="cuda")
        return x.to(stored)

    serve = case["mode"] == "serve"
    inputs = [image_batch(b) for b in (batches(case) if serve else [case["batch"]])]
    outs = []
    for i, (fam, model) in enumerate(zip(fams, models)):
        blob = weights(model, seed * 64 + i + 1, tiny).cuda()
        x = inputs[i if serve else 0].double().permute(0, 3, 1, 2)
        outs.append(torch.cat([forward64(model, blob, part) for part in x.split(8)]).float())
    return outs


def activation64(y, act):
    if act == zoo.RELU:
        return y.clamp(min=0)
    if act == zoo.RELU6:
        return y.clamp(0, 6)
    gates = {zoo.HARDSWISH: lambda v: v * (v + 3).clamp(0, 6) / 6, zoo.HARDSIGMOID: lambda v: (v + 3).clamp(0, 6) / 6,
             zoo.SILU: lambda v: v * torch.sigmoid(v), zoo.SIGMOID: torch.sigmoid, zoo.NONE: lambda v: v}
    return gates[act](y)


def forward64(model, blob, x):
    """One model in 64 bits on an NCHW batch; a layer's value is dropped after its last reader."""
    stored, size = (torch.float32, 4) if model.dtype == "f32" else (torch.bfloat16, 2)
    last = {}
    for i, layer in enumerate(model.layers):
        last[layer.input] = last[layer.residual] = i
    values = {zoo.MODEL_INPUT: x}
    for i, layer in enumerate(model.layers):
        v, n = values[layer.input], x.shape[0]
        other = values.get(layer.residual)
        kh, kw = layer.k, layer.kw or layer.k
        if layer.op in (zoo.CONV, zoo.DWCONV, zoo.FC):
            groups = {zoo.CONV: layer.groups, zoo.DWCONV: layer.cout, zoo.FC: 1}[layer.op]
            if layer.op == zoo.FC:
                v, kh, kw, stride, pad = v.reshape(n, layer.cin, 1, 1), 1, 1, 1, 0
            else:
                stride = layer.stride
                pad = layer.pad if kh == kw else (layer.pad if kh > 1 else 0, layer.pad if kw > 1 else 0)
            count = layer.cout * (v.shape[1] // groups) * kh * kw
            w = blob[layer.w_off:layer.w_off + count * size].view(stored).double().view(groups, layer.cout // groups, -1)
            b = blob[layer.b_off:layer.b_off + 4 * layer.cout].view(torch.float32).double()
            y = torch.empty((n, layer.cout, layer.out_h, layer.out_w), dtype=torch.float64, device=x.device)
            for image in range(n):
                taps = torch.nn.functional.unfold(v[image:image + 1].contiguous(), (kh, kw), padding=pad, stride=stride)
                y[image] = torch.matmul(w, taps.view(groups, w.shape[2], -1)).view(y.shape[1:])
            y += b.view(1, -1, 1, 1)
            y = activation64(y if other is None else y + other, layer.act)
        elif layer.op == zoo.MAXPOOL:
            y = torch.nn.functional.max_pool2d(v, kh, layer.stride, layer.pad, ceil_mode=layer.ceil)
        elif layer.op == zoo.AVGPOOL:
            y = torch.nn.functional.avg_pool2d(v, kh, layer.stride, layer.pad)
        elif layer.op == zoo.GAP:
            y = v.mean((2, 3), keepdim=True)
        elif layer.op == zoo.SOFTMAX:
            y = torch.softmax(v, 1)
        elif layer.op == zoo.CONCAT:
            y = torch.cat([v, other], 1)
        elif layer.op == zoo.MUL:
            y = v * other
        elif layer.op == zoo.SLICE:
            y = v[:, layer.first:layer.first + layer.cout]
        else:   # shuffle: the channels as a groups x rest matrix, transposed
            y = v.view(n, layer.groups, -1, *v.shape[2:]).transpose(1, 2).reshape(v.shape)
        values[i] = y
        for done in [k for k in values if last.get(k, i) <= i and k != i]:
            del values[done]
    return values[model.output].reshape(x.shape[0], -1)


def work(case):
    """Images and weights in once, logits out once; two operations per multiply-add."""
    size = 4 if case["dtype"] == "f32" else 2
    own = batches(case)
    fams = families(case)
    models = {fam: model_of(case, fam) for fam in set(fams)}
    images = sum(own) if case["mode"] == "serve" else case["batch"]
    nbytes = images * case["side"] ** 2 * 3 * size
    for fam, b in zip(fams, own):
        nbytes += models[fam].n_params() * size + b * models[fam].layers[-1].cout * 4
    return {"bytes": nbytes, "flops": 2 * multiply_adds(case)}


def tolerance(case):
    fams = set(families(case))
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 4e-5}
    if fams <= WIDE:
        return {"rel": 1e-4, "max": 4e-4}
    return {"rel": 2.4e-2, "max": 8e-2} if fams & ROUGH else {"rel": 1.4e-2, "max": 5e-2}
