"""What a user of this library has it do, as cases that can be timed and compared.

Four kinds of work, each through the public entry points (`paper_1909_11985_amd.binding`):

  step      one synchronous mini-batch of an elastic job (`Job.step`): shard assignment, gather, forward and
            backward of the p workers' shards, aggregation and update
  update    aggregation + update on the caller's own arrays (`edl_average_update`, `edl_adam_update`)
  join      the state image an adjustment hands to a joining worker (`Job.snapshot`, then `Job.restore` there)
  shard     one mini-batch's sample assignment from (seed, epoch, step) on the host (`edl_shard_host`)

Sizes are those of the repository's configurations, benchmark and tests, and of the networks it names.
"""
import math

import numpy as np
import torch

import paper_1909_11985_amd.binding as edl

# image height, width, channels and classes of a model's default job
DEFAULTS = {"mlp": (1, 784, 10), "resnet20": (32, 3, 10), "resnet50": (224, 3, 1000), "vgg16": (224, 3, 1000),
            "alexnet": (224, 3, 1000)}
LR = {"mlp": 0.1, "resnet20": 0.1, "resnet50": 0.1, "vgg16": 0.001, "alexnet": 0.001}
# Size of the momentum a job has in mid-training: a few times the size of its gradients.
MOMENTUM_SIZE = {"mlp": 0.05, "resnet20": 0.02, "resnet50": 0.02, "vgg16": 0.05, "alexnet": 0.05}


def listed():
    return [
        # the smallest job: a fully connected net in four shards of 16; launches and host work
        dict(name="mlp_f32_b64_p4", kind="step", model="mlp", dtype="f32", B=64, p=4),
        # a small residual net at the far end of its 2 -> 4 -> 8 schedule, the loss read back at every step
        dict(name="resnet20_f32_b128_p8", kind="step", model="resnet20", dtype="f32", B=128, p=8, loss=True),
        # the headline job: one worker's shard of 32
        dict(name="resnet50_bf16_b32_p1", kind="step", model="resnet50", dtype="bf16", B=32, p=1),
        # the elastic job (aggregate batch 256, any p from 1 to 8) while it runs on eight workers: the largest
        dict(name="resnet50_bf16_b256_p8", kind="step", model="resnet50", dtype="bf16", B=256, p=8, max_shard=256),
        # a mini-batch of 64 redone by three survivors of four (22 + 21 + 21), images of an odd size
        dict(name="resnet50_bf16_b64_p3_uneven", kind="step", model="resnet50", dtype="bf16", B=64, p=3, image=161, uneven=True),
        # the large dense net: long contractions, 138 M parameters to update
        dict(name="vgg16_bf16_b32_p1", kind="step", model="vgg16", dtype="bf16", B=32, p=1),
        # two workers' shards of 64, fully connected layers and Adam over 61 M parameters
        dict(name="alexnet_bf16_b128_p2_adam", kind="step", model="alexnet", dtype="bf16", B=128, p=2, optimizer="adam"),
        # aggregation + update alone: a small float32 state and an odd number of workers
        dict(name="update_f32_272k_p3", kind="update", P=272474, p=3, bf16=False),
        # ... the largest state, four workers, with the bf16 copy
        dict(name="update_bf16_138m_p4", kind="update", P=138357544, p=4, bf16=True),
        # ... Adam, eight workers of unequal shares
        dict(name="adam_bf16_26m_p8_shares", kind="update", P=25557032, p=8, bf16=True, optimizer="adam", shares=True),
        # a scale-out: the state image taken and restored into the joiner
        dict(name="join_resnet50", kind="join", model="resnet50", dtype="bf16", B=32, p=1),
        # the assignment of one mini-batch of an epoch over 1.2 million samples
        dict(name="shard_1200k", kind="shard", N=1200000, B=250, p=10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_model(rng):
    """A job of one of the models: the network's depth, the image and the shard over the range they are run in."""
    model = rng.choice(["mlp", "resnet20", "resnet50", "resnet50", "vgg16", "alexnet"])
    c = dict(model=model, p=rng.choice([1, 2, 3, 4, 5, 8]))
    if model == "mlp":
        shard = _log_int(rng, 8, 512)
        c.update(dtype=rng.choice(["f32", "bf16"]), arch="%d,%d" % (_log_int(rng, 64, 1024), _log_int(rng, 64, 1024)))
    elif model == "resnet20":
        shard = min(_log_int(rng, 8, 256), 512 // c["p"])
        c.update(dtype="f32", image=rng.randint(24, 40))
    elif model == "resnet50":
        c.update(dtype="bf16", image=rng.randint(112, 224), arch=rng.choice(["64,3,4,6,3", "64,3,4,6,3", "64,3,4,23,3"]))
        cost = (c["image"] / 224.0) ** 2 * (2.0 if "23" in c["arch"] else 1.0)
        shard = max(8, min(_log_int(rng, 8, 128), int(200 / cost / c["p"])))
    elif model == "vgg16":
        c.update(dtype="bf16", image=rng.randint(64, 224), p=min(c["p"], 4), arch=rng.choice(["64,4096,2,2,3,3,3", "64,1024,2,2,3,3,3", "64,1024,2,2,4,4,4"]))
        shard = max(4, min(_log_int(rng, 4, 64), int(64 / (c["image"] / 224.0) ** 2 / c["p"])))
    else:
        shard = min(_log_int(rng, 16, 256), 512 // c["p"])
        c.update(dtype="bf16", image=rng.randint(96, 224), arch=rng.choice(["64,4096", "64,1024"]))
    c["B"] = c["p"] * shard
    if rng.random() < 0.25:
        c["optimizer"] = "adam"
    return c


def draw(rng):
    kind = rng.choice(["step"] * 8 + ["update"] * 2 + ["join", "shard"])
    if kind == "step":
        c = dict(kind=kind, **_draw_model(rng))
        if c["p"] > 1 and rng.random() < 0.25:
            # the next larger worker count's mini-batch, redone by p of its workers
            c["B"] += rng.randint(1, c["p"] - 1)
            c["uneven"] = True
        if rng.random() < 0.25:
            c["loss"] = True
        return c
    if kind == "update":
        c = dict(kind=kind, P=_log_int(rng, 20000, 138357544), p=rng.choice([1, 2, 3, 4, 5, 8]), bf16=rng.random() < 0.7)
        if rng.random() < 0.4:
            c.update(optimizer="adam", shares=rng.random() < 0.3)
        return c
    if kind == "join":
        return dict(kind=kind, **_draw_model(rng))
    B = _log_int(rng, 16, 1024)
    return dict(kind=kind, N=B * _log_int(rng, 4, 2000000 // B), B=B, p=1)


# ---------------------------------------------------------------------------------------------------- preparation
def _config(case):
    model = case["model"]
    image, channels, classes = DEFAULTS[model]
    image = case.get("image", image)
    B, p = case["B"], case["p"]
    arch = tuple(int(a) for a in case["arch"].split(",")) if "arch" in case else ()
    # data set: a few mini-batches, so that epochs end and new permutations are drawn
    return edl.make_config(model, dtype=case["dtype"], N=4 * B, B=B, p_max=p, max_shard=case.get("max_shard", -(-B // p)),
                           lr=LR[model] if case.get("optimizer") != "adam" else 1e-3, H=image, W=image, C_=channels, classes=classes,
                           arch=arch, optimizer=case.get("optimizer", "momentum"))


def _job(case, seed, rng):
    """A job in mid-training: He-initialised weights, non-zero momentum, residual blocks whose last batch norm has a
    small scale (they are started at zero in large-batch training; at scale 1 a bf16 residual net's gradient is set by
    rounding, so that no two correct implementations would agree on it), and for the nets without batch norm logits of
    order one (at He-initialised weights they start near 15)."""
    cfg = _config(case)
    job = edl.Job(cfg, seed)
    P = job.sizes.P
    image = job.snapshot()
    state = image[256:].view(torch.float32)
    last = {"resnet20": ".bn2.g", "resnet50": ".bn3.g", "vgg16": "fc3.w", "alexnet": "fc3.w"}.get(case["model"])
    for name, off, size, _ in edl.edl_tensor_table(cfg):
        if last is None or not name.endswith(last):
            continue
        if last == "fc3.w":
            state[off:off + size].mul_(0.1)
        else:
            state[off:off + size].uniform_(0.0, 0.01, generator=rng)
    state[P:2 * P].normal_(0.0, MOMENTUM_SIZE[case["model"]], generator=rng)
    if case.get("optimizer") == "adam":
        state[2 * P:3 * P].uniform_(0.5, 2.0, generator=rng).mul_(MOMENTUM_SIZE[case["model"]] ** 2)
    job.restore(image)
    return job


def _views(job):
    """The job's own state arrays."""
    s, a = job.sizes, job.arena
    out = {"w": a[s.params_off:s.params_off + 4 * s.P].view(torch.float32),
           "v": a[s.momentum_off:s.momentum_off + 4 * s.P].view(torch.float32)}
    if s.second_off >= 0:
        out["s"] = a[s.second_off:s.second_off + 4 * s.P].view(torch.float32)
    if s.R:
        out["running"] = a[s.running_off:s.running_off + 4 * s.R].view(torch.float32)
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "shard":
        return dict(case=case, seed=seed, epoch=seed % 7, step=seed % (case["N"] // case["B"]))
    rng = torch.Generator(device="cuda").manual_seed(seed)
    if kind == "update":
        P, p = case["P"], case["p"]
        st = dict(case=case, grads=[torch.randn(P, device="cuda", generator=rng).mul_(1e-2) for _ in range(p)],
                  w=torch.randn(P, device="cuda", generator=rng).mul_(0.05), v=torch.randn(P, device="cuda", generator=rng).mul_(0.05),
                  w16=torch.empty(P, device="cuda", dtype=torch.bfloat16) if case["bf16"] else None, shares=None)
        if case.get("optimizer") == "adam":
            st["s"] = torch.rand(P, device="cuda", generator=rng).add_(0.5).mul_(1e-4)
            if case.get("shares"):
                n = np.arange(p) + 20.0
                st["shares"] = (n / n.sum()).tolist()
        return st
    job = _job(case, seed, rng)
    if kind == "join":
        return dict(case=case, job=job, joiner=edl.Job(_config(case), seed + 1),
                    image=torch.empty(job.sizes.snapshot_bytes, dtype=torch.uint8, device="cuda"))
    cfg = job.cfg
    x = torch.randn(cfg.N, cfg.H, cfg.W, cfg.C, device="cuda", generator=rng)
    y = torch.randint(0, cfg.classes, (cfg.N,), device="cuda", dtype=torch.int32, generator=rng)
    job.bind_dataset(x, y)
    st = dict(case=case, job=job, state=_views(job))
    if case.get("uneven"):
        B, p = case["B"], case["p"]
        st["off"] = np.concatenate([[0], np.cumsum([B // p + (k < B % p) for k in range(p)])]).astype(np.int64)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "step":
        job, want = st["job"], case.get("loss", False)
        if case.get("uneven"):
            _, epoch, step = job.progress()
            idx, _ = job.shard(case["B"], 1, epoch, step)
            loss = job.step(case["p"], idx, st["off"], want_loss=want)
        else:
            loss = job.step(case["p"], want_loss=want)
        return dict(st["state"], loss=loss) if want else st["state"]
    if kind == "update":
        if case.get("optimizer") == "adam":
            edl.edl_adam_update(st["grads"], st["w"], st["v"], st["s"], st["w16"], 1e-3, 0.9, 0.999, 1e-8, 5e-4, 10, shares=st["shares"])
            return dict(w=st["w"], v=st["v"], s=st["s"], w16=st["w16"])
        edl.edl_average_update(st["grads"], st["w"], st["v"], st["w16"], 0.01, 0.9, 5e-4)
        return dict(w=st["w"], v=st["v"], w16=st["w16"])
    if kind == "join":
        st["job"].snapshot(st["image"])
        st["joiner"].restore(st["image"])
        return dict(_views(st["joiner"]), image=st["image"])
    idx, off = edl.edl_shard_host(st["seed"], case["N"], case["B"], case["p"], st["epoch"], st["step"])
    st["step"] += 1
    if st["step"] == case["N"] // case["B"]:
        st["step"], st["epoch"] = 0, st["epoch"] + 1
    return dict(idx=idx, off=off)


# ------------------------------------------------------------------------------------------------ work, tolerance
def work(case):
    """Bytes every pass must move (inputs read once, outputs written once) and its contractions' flops."""
    kind, adam = case["kind"], case.get("optimizer") == "adam"
    if kind == "shard":
        return {"bytes": 8.0 * case["N"], "flops": 0.0}          # the epoch's permutation
    if kind == "update":
        return {"bytes": (4.0 * case["p"] + (24.0 if adam else 16.0) + (2.0 if case["bf16"] else 0.0)) * case["P"], "flops": 0.0}
    cfg = _config(case)
    s = edl.edl_query(cfg)
    slots = 3 if adam else 2
    if kind == "join":
        return {"bytes": 4.0 * s.snapshot_bytes, "flops": 0.0}    # state read, image written; image read, state written
    return {"bytes": 4.0 * case["B"] * cfg.H * cfg.W * cfg.C + 8.0 * slots * s.P + (2.0 * s.P if case["dtype"] == "bf16" else 0.0),
            "flops": s.flops_per_sample * case["B"]}


def tolerance(case):
    kind = case["kind"]
    if kind in ("join", "shard"):
        return "exact"
    if kind == "update":
        # float32 sums of p terms in any order; the bf16 copy may round to the neighbour where w differs
        return {"rel": 1e-5 if not case["bf16"] else 1e-4, "max": 1e-2}
    if case["dtype"] == "f32":
        # float32 sums in another order, and the occasional pre-activation near 0 that takes the other sign
        return {"rel": 1e-3, "max": 0.1}
    # bf16 activations and gradients through up to a hundred layers
    return {"rel": 1e-2, "max": 0.9}
