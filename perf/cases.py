"""Performance cases of the library: the calls that a user's program makes, with their inputs.

`listed()` names the fixed cases, `draw(rng)` gives one more of the same ranges.  A case says which procedure
runs (certification, prediction, a batch of either, a comparison system, a stored noise bank), on which of the
synthetic networks, at which sizes.  `prepare` makes the model handle, its workspace and the images, `run` is one
call of the procedure.

The synthetic networks have random weights, whose class means lie so far apart that every noisy copy gets the
same vote.  `prepare` therefore loads them with the bias of the last layer centred on the mean logits of one
reference image, as a trained network's are near a decision boundary: the votes split and depend on every layer.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2108_09413_amd as isr
import synth

ALPHA = 0.001
# workload configuration and device chunk (noisy copies) of each network, as bench.py runs them
NETS = {"tiny": (0, 1024), "resnet20": (1, 8192), "resnet110": (2, 4096), "resnet50": (3, 668)}
# most inferences of a drawn case: none costs more than the largest listed one
MOST_INFERENCES = {"tiny": 100000, "resnet20": 100000, "resnet110": 100000, "resnet50": 100000}
MOST_FP_INFERENCES = {"tiny": 100000, "resnet20": 100000, "resnet110": 20000, "resnet50": 4000}


def listed():
    return [
        # Alg. 2 at the smallest sample size of the evaluation: one call per image, where launches and latency count
        dict(name="predict-resnet20-n100", do="predict", net="resnet20", size=32, chunk=8192, sigma=64, n=100),
        # workload configuration 0: a small certification of the two-convolution net
        dict(name="certify-tiny-n1000", do="certify", net="tiny", size=32, chunk=1024, sigma=32, n0=100, n=1000),
        # configuration 1: CIFAR-shaped certification at the paper's N
        dict(name="certify-resnet20-n100k", do="certify", net="resnet20", size=32, chunk=8192, sigma=32, n0=100, n=100000),
        # configuration 2: the deep CIFAR-shaped net
        dict(name="certify-resnet110-n100k", do="certify", net="resnet110", size=32, chunk=4096, sigma=64, n0=100, n=100000),
        # Alg. 2 on the large net, one image at a time: a chunk that is far from full
        dict(name="predict-resnet50-n100", do="predict", net="resnet50", size=224, chunk=668, sigma=64, n=100),
        # configuration 3: Caltech-101-shaped certification
        dict(name="certify-resnet50-n10k", do="certify", net="resnet50", size=224, chunk=668, sigma=128, n0=100, n=10000),
        # configuration 4: the headline workload and the largest case
        dict(name="certify-resnet50-n100k", do="certify", net="resnet50", size=224, chunk=668, sigma=64, n0=100, n=100000),
        # a sweep of the evaluation: many (image, sigma) pairs with few samples each in one call
        dict(name="predict-batch-resnet20", do="predict_batch", net="resnet20", size=32, chunk=8192, sigma=64, items=256, images=64,
             sigmas=3, n=100),
        # certification of several images at several noise levels with an odd number of samples per pair
        dict(name="certify-batch-resnet50", do="certify_batch", net="resnet50", size=224, chunk=668, sigma=32, items=7, images=5,
             sigmas=4, n0=50, n=777),
        # noise stored ahead of training for a whole CIFAR-shaped training set
        dict(name="noise-bank-50000x3072", do="noise_bank", sigma=32, count=50000, d=3072),
        # the fp32 comparison system (Efficiency Evaluation) on the large net
        dict(name="floatrs-fp-resnet50", do="float", system="fp", net="resnet50", size=224, chunk=2672, sigma=64, n0=100, n=4000),
        # the comparison system that shares the int8 network
        dict(name="floatrs-quant-resnet20", do="float", system="quant", net="resnet20", size=32, chunk=8192, sigma=32, n0=100,
             n=10000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["certify", "certify", "predict", "predict", "predict_batch", "certify_batch", "float", "noise_bank"])
    sigma = _log_int(rng, 16, 256)
    if do == "noise_bank":
        # from one training batch to a whole set; any noise level that the sampler takes
        d = rng.choice([784, 3072, 4 * rng.randrange(200, 3000), 3 * 64 * 64, 3 * 224 * 224])
        return dict(do=do, sigma=_log_int(rng, 1, 1024), count=_log_int(rng, 16, max(17, min(50000, 150_000_000 // d))), d=d)
    net = rng.choice(["tiny", "resnet20", "resnet20", "resnet110", "resnet50", "resnet50", "resnet50"])
    # other input sizes than 224 give feature maps whose sides are odd or divide no tile
    size = rng.choice([224, 224, 224, 96, 128, 160, 192]) if net == "resnet50" else 32
    full = NETS[net][1]
    chunk = rng.choice([full, full, _log_int(rng, full // 4, full)])
    most = MOST_INFERENCES[net]
    case = dict(do=do, net=net, size=size, chunk=chunk, sigma=sigma)
    if do == "certify":
        case.update(n0=rng.choice([100, 100, rng.randrange(20, 300)]), n=_log_int(rng, 1000, most - 300))
    elif do == "predict":
        case.update(n=_log_int(rng, 20, most // 10))
    elif do == "float":
        case["system"] = rng.choice(["fp", "quant"])
        if case["system"] == "fp":
            most = MOST_FP_INFERENCES[net]
            case["chunk"] = 4 * chunk   # fp32 tensors take four times the bytes
        case.update(n0=100, n=_log_int(rng, 500, min(most, 20000)))
    else:
        images = rng.randrange(2, 12)
        items = _log_int(rng, 4, 200)
        per = _log_int(rng, 50, max(60, min(2000, most // 2 // items)))
        case.update(items=items, images=images, sigmas=rng.randrange(1, 7), n=per)
        if do == "certify_batch":
            case.update(n0=rng.randrange(20, 120))
    return case


@functools.lru_cache(maxsize=None)
def _net_blob(net, size, sigma):
    """The network as a user keeps it on disk: synthetic weights, last bias centred (module docstring)."""
    config = NETS[net][0]
    blob = synth.build_model(config, size=size)
    classes = synth.CONFIGS[config]["classes"]
    model = isr.isr_load_model(blob)
    isr.isr_set_workspace(model, 64)
    image = synth.make_image(config, 1, shape=(3, size, size))
    logits = isr.isr_debug_forward(model, image, sigma, 1, 1, 0, 0, 64)[0]
    model.close()
    # the last operation's payload ends with the bias, int32 [classes]
    bias = np.frombuffer(blob[-4 * classes:], dtype="<i4") - np.rint(logits.mean(axis=0)).astype("<i4")
    return blob[:-4 * classes] + bias.astype("<i4").tobytes()


def _images(seed, count, size):
    """uint8 [count][3][size][size]: smooth random fields over the full range, as photographs quantised to 8 bits."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.rand((count, 3, size + 2, size + 2), generator=g, device="cuda")
    x = 0.25 * x[:, :, :-2] + 0.5 * x[:, :, 1:-1] + 0.25 * x[:, :, 2:]
    x = 0.25 * x[..., :-2] + 0.5 * x[..., 1:-1] + 0.25 * x[..., 2:]
    lo, hi = x.amin(dim=(1, 2, 3), keepdim=True), x.amax(dim=(1, 2, 3), keepdim=True)
    return torch.round((x - lo) / (hi - lo) * 255.0).to(torch.uint8).contiguous()


def prepare(case, seed):
    if case["do"] == "noise_bank":
        return dict(case=case, seed=seed, out=torch.empty((case["count"], case["d"]), dtype=torch.int16, device="cuda"))
    model = isr.isr_load_model(_net_blob(case["net"], case["size"], case["sigma"]))
    isr.isr_set_workspace(model, case["chunk"], float_fp=case.get("system") == "fp")
    state = dict(case=case, seed=seed, model=model, images=_images(seed, case.get("images", 1), case["size"]))
    state["image"] = state["images"][0]
    if "items" in case:
        # the sweep's pairs: images in turn, noise levels around the base one (at most 8 of them)
        levels = [min(1024, max(1, case["sigma"] + 3 * k)) for k in range(case["sigmas"])]
        state["items"] = [(i % case["images"], levels[(i // case["images"]) % len(levels)], i % case["images"] + 1)
                          for i in range(case["items"])]
    return state


def _one(res, *votes):
    return dict(cls=res.cls, radius=res.radius, p_lower=res.p_lower, n_top=res.n_top, n_second=res.n_second,
                radius_int=res.radius_int, radius_sq_int=res.radius_sq_int, votes=list(votes))


def _many(results, *votes):
    return dict(cls=np.array([r.cls for r in results]), radius=np.array([r.radius for r in results]),
                p_lower=np.array([r.p_lower for r in results]), votes=list(votes))


def run(state):
    c, seed = state["case"], state["seed"]
    if c["do"] == "certify":
        return _one(*isr.isr_certify(state["model"], state["image"], c["sigma"], c["n0"], c["n"], ALPHA, seed=seed, image_id=1))
    if c["do"] == "predict":
        return _one(*isr.isr_predict(state["model"], state["image"], c["sigma"], c["n"], ALPHA, seed=seed, image_id=1))
    if c["do"] == "certify_batch":
        return _many(*isr.isr_certify_batch(state["model"], state["images"], state["items"], c["n0"], c["n"], ALPHA, seed=seed))
    if c["do"] == "predict_batch":
        return _many(*isr.isr_predict_batch(state["model"], state["images"], state["items"], c["n"], ALPHA, seed=seed))
    if c["do"] == "noise_bank":
        return isr.isr_noise_bank(c["sigma"], seed, 1, 0, c["count"], c["d"], out=state["out"])
    system = isr.FLOATRS_FP if c["system"] == "fp" else isr.FLOATRS_QUANT
    res, votes0, votes1 = isr.isr_float_certify(state["model"], state["image"], float(c["sigma"]), c["n0"], c["n"], ALPHA, system,
                                                seed=seed, image_id=1)
    if system == isr.FLOATRS_QUANT:
        return _one(res, votes0, votes1)
    # fp32 logits are reproducible up to the rounding of their sums: a copy whose two best classes tie within it may
    # vote either way, so the tallies count as measured values (float64), not as whole numbers
    return dict(p_lower=res.p_lower, votes=np.stack([votes0, votes1]).astype(np.float64))


@functools.lru_cache(maxsize=None)
def _macs_and_bytes(net, size):
    config = NETS[net][0]
    return synth.model_macs(config, size=size), len(synth.build_model(config, size=size))


def _inferences(case):
    return (case.get("n0", 0) + case["n"]) * case.get("items", 1)


def work(case):
    """Two operations per multiply-accumulate of every inference; the weights and the images read once (activations
    need not leave the chip); for a noise bank the draws written."""
    if case["do"] == "noise_bank":
        return dict(bytes=2 * case["count"] * case["d"], flops=0)
    macs, weight_bytes = _macs_and_bytes(case["net"], case["size"])
    scale = 4 if case.get("system") == "fp" else 1
    return dict(bytes=scale * weight_bytes + case.get("images", 1) * 3 * case["size"] ** 2, flops=2 * macs * _inferences(case))


def tolerance(case):
    if case["do"] == "noise_bank":
        return "exact"
    if case.get("system") == "fp":
        # a few copies in a near tie (see run); one moves two tallies by 1
        return dict(rel=min(0.03, max(2e-3, 8.0 / case["n"])))
    # tallies and classes are whole numbers and exact; radius and bound are float64 functions of them
    return dict(rel=1e-9)
