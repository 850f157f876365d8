"""What a user of this framework has it do, as timed cases.

A case is one network, registered through ``GraphRunner``, put through the ahead-of-time pass once
(``prepare``) and replayed (``run``) in the default mode, ``NG_MODE_AUTO``. One pass is what ``bench.py``
times: replay, wait, and the results are there. The networks are the recipes of ``workloads``; the
topology and the weights are those of the recipes' default seed, as a program keeps one network, and the
input tensors (and dL/d(output) of a training step) come from the seed of ``prepare``.
"""
import dataclasses
import functools

import numpy as np
import torch

import workloads
from paper_2012_02732_amd import GraphRunner
from paper_2012_02732_amd import binding as B

DEVICE = "cuda:0"
LEARNING_RATE = 1e-6          # small, so that thousands of passes on one state leave the weights in their range


def listed():
    return [
        # the smallest network anybody runs: seven tasks, the cost of a call is launching it and waiting for it
        {"name": "tiny_cell", "net": "tiny"},
        # a plain chain of small 3 x 3 convolutions: no task can run beside another
        {"name": "chain50", "net": "chain", "blocks": 50},
        # wide random DAG of 200 small tasks (adds, channel slices, 1 x 1 and depthwise convolutions)
        {"name": "random200", "net": "random", "nodes": 200, "channels": 64, "size": 28},
        # interactive inference with a searched network: one image, 483 tasks of 1-3 us
        {"name": "nasnet_b1", "net": "nasnet", "cells": 4, "channels": 44, "image": 224, "host": False},
        # the same from a program that has its images in host memory and wants the scores there
        {"name": "nasnet_b1_host", "net": "nasnet", "cells": 4, "channels": 44, "image": 224, "host": True},
        # an image size that leaves odd maps everywhere (25 x 25, 13 x 13, 7 x 7)
        {"name": "nasnet_b1_odd", "net": "nasnet", "cells": 4, "channels": 44, "image": 193, "host": False},
        # a hand-designed network with large convolutions: one image, a small ragged batch, a full batch
        {"name": "inception_b1", "net": "inception", "batch": 1, "image": 299, "host": False},
        {"name": "inception_b6_odd", "net": "inception", "batch": 6, "image": 261, "host": False},
        {"name": "inception_b32", "net": "inception", "batch": 32, "image": 299, "host": False},
        # training steps (forward, backward, SGD update as one DAG) on CIFAR-sized images: the usual batch,
        # a small batch of odd images, a large batch
        {"name": "train_b32", "net": "train", "batch": 32, "channels": 44, "image": 32},
        {"name": "train_b10_odd", "net": "train", "batch": 10, "channels": 36, "image": 27},
        {"name": "train_b96", "net": "train", "batch": 96, "channels": 44, "image": 32},
    ]


def _spread(rng, lo, hi):
    """A whole number from lo to hi, uniform in its logarithm."""
    return min(hi, int(lo * (hi / lo) ** rng.random() + 0.5))


def draw(rng):
    net = rng.choice(["chain", "random", "nasnet", "nasnet", "inception", "inception", "train", "train"])
    if net == "chain":
        return {"net": net, "blocks": _spread(rng, 8, 100)}
    if net == "random":
        return {"net": net, "nodes": rng.randint(60, 240), "channels": rng.randint(16, 96), "size": rng.randint(7, 56)}
    if net == "nasnet":
        return {"net": net, "cells": rng.randint(2, 5), "channels": rng.choice([24, 32, 36, 44, 52, 64]),
                "image": rng.randint(128, 320), "host": rng.random() < 0.25}
    if net == "inception":
        return {"net": net, "batch": _spread(rng, 1, 32), "image": rng.randint(139, 299), "host": False}
    batch = _spread(rng, 4, 128)
    return {"net": net, "batch": batch, "channels": rng.choice([24, 32, 36, 44, 48]), "image": rng.randint(12, 36)}


@functools.lru_cache(maxsize=4)
def _network(**case):
    net = case["net"]
    if net == "tiny":
        return workloads.make("tiny_cell")
    if net == "chain":
        return workloads.make("chain50", blocks=case["blocks"])
    if net == "random":
        return workloads.make("random200", n_nodes=case["nodes"], shape=(1, case["channels"], case["size"], case["size"]))
    if net == "nasnet":
        return workloads.make("nasnet_style", cells_per_stage=case["cells"], c0=case["channels"], image=case["image"])
    if net == "inception":
        return workloads.make("inception_style", batch=case["batch"], image=case["image"])
    return workloads.nas_cell_cifar(batch=case["batch"], c=case["channels"], image=case["image"])


def _net_of(case):
    return _network(**{k: v for k, v in case.items() if k not in ("name", "host")})


@dataclasses.dataclass
class State:
    runner: GraphRunner
    image: np.ndarray             # a host caller's image
    host: bool
    results: dict                 # tensors a caller on the GPU reads after a pass: views of the arena and the weights


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    net = _net_of(case)
    image = rng.standard_normal(net.input.shape, dtype=np.float32)
    w = dataclasses.replace(net, input=image)
    if case["net"] == "train":
        out = net.outputs[0]
        gradient = rng.standard_normal(net.nodes[out].shape, dtype=np.float32) / net.nodes[out].shape[0]
        w = workloads.training_graph(w, LEARNING_RATE, {out: gradient})
    r = GraphRunner(w, DEVICE)
    r.prepare()
    base = r.arena.data_ptr()

    def tensor(v):
        shape = B.ng_node_shape(r.g, v)
        at = B.ng_tensor_ptr(r.g, v) - base
        return r.arena[at:at + 4 * int(np.prod(shape))].view(torch.float32).view(*shape)

    if case["net"] == "train":
        results = {"logits": tensor(net.outputs[0])}
        for v in sorted({node for node, _, _ in w.wgrad_of.values()}):
            results["gradient %d" % v] = tensor(v)                       # of every weight of the network
        for v, nd in enumerate(net.nodes):
            if nd.op in ("conv3x3", "dwconv", "fc"):
                for j in range(len(nd.weights)):
                    results["weight %d %d" % (v, j)] = r._weights[(v, j)]  # updated in place
    else:
        # a wide random DAG has more sinks than anybody reads at once: the last ones, which hang on everything before
        results = {"output %d" % v: tensor(v) for v in w.outputs[-64:]}
    return State(r, image, bool(case.get("host")), results)


def run(state):
    if state.host:
        return state.runner.run(state.image)
    state.runner.replay()
    state.runner.sync()
    return state.results


def _flops(net):
    total = [0.0] * len(net.nodes)
    for v, nd in enumerate(net.nodes):
        out = float(np.prod(nd.shape))
        cin = net.nodes[nd.preds[0]].shape[1] if nd.preds else 0
        if nd.op in ("conv1x1", "fc"):
            total[v] = 2 * cin * out
        elif nd.op == "conv3x3":
            total[v] = 18 * cin * out
        elif nd.op == "dwconv":
            total[v] = 2 * nd.params["k"] ** 2 * out
        elif nd.op == "pool":
            total[v] = 9 * out
        elif nd.op in ("bn_act", "add_n", "relu"):
            total[v] = 2 * out
        elif nd.op == "global_avgpool":
            total[v] = float(np.prod(net.nodes[nd.preds[0]].shape))
    return total


def work(case):
    """Input and weights read once, results written once; a training step also writes every gradient and every
    updated weight, and its backward pass takes two products where the forward pass takes one."""
    net = _net_of(case)
    weights = sum(w.size for nd in net.nodes for w in nd.weights)
    values = net.input.size + weights + sum(float(np.prod(net.nodes[o].shape)) for o in net.outputs)
    flops = sum(_flops(net))
    if case["net"] == "train":
        values += 2 * weights + float(np.prod(net.nodes[net.outputs[0]].shape))
        flops *= 3
    return {"bytes": 4.0 * values, "flops": flops}


def tolerance(case):
    """About four times what separates the path from the same network in 64 bits, where no decision changes. In a
    training step rounding also decides ties: an element whose ReLU mask or max-pool tap flips moves a gradient's
    norm by up to 3e-3 and its largest element by 2e-2 of the root mean square (seen against 64 bits)."""
    if case["net"] == "train":
        return {"rel": 1.2e-2, "max": 7e-2}
    if case["net"] == "chain":
        return {"rel": 2e-5, "max": 2e-4}
    return {"rel": 3e-6, "max": 3e-5}
