"""CPU-only checks of the C boundary: the library loads, exports every symbol
the header declares, and its host logic (shard assignment, initialisation,
parameter layout) agrees with the oracle.  No compute call is made."""
import os
import re

import numpy as np
import pytest

from oracle import oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def E():
    import paper_1909_11985_amd as E
    return E


def test_every_declared_symbol_is_exported(E):
    text = open(os.path.join(ROOT, "include", "edl.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = set(re.findall(r"\b(edl_[a-z0-9_]+)\s*\(", text))
    assert len(declared) >= 20
    for name in sorted(declared):
        assert hasattr(E.lib, name), name
    from paper_1909_11985_amd import binding
    assert declared == set(binding.EXPORTS)


@pytest.mark.parametrize("seed", [0, 7, 2**63 + 5])
@pytest.mark.parametrize("N,B", [(64, 8), (1024, 64), (2048, 128), (2048, 256)])
def test_shard_assignment_is_bit_exact(E, seed, N, B):
    for epoch in (0, 1, 5):
        for t in (0, N // B - 1):
            for p in (1, 2, 4, 8):
                idx, off = E.edl_shard_host(seed, N, B, p, epoch, t)
                io, oo = O.shard(seed, N, B, p, epoch, t)
                assert idx.dtype == np.int64 and np.array_equal(idx, io) and np.array_equal(off, oo)


@pytest.mark.parametrize("N,B", [(4096, 1), (65536, 16), (100000, 250), (262144, 512), (500000, 1000), (1 << 20, 64)])
def test_shard_assignment_by_followed_entries(E, N, B):
    """Mini-batches that are a small part of a large data set are not walked to but followed back: every part of the epoch,
    its first and last mini-batch, against the whole permutation."""
    steps = N // B
    for epoch in (0, 3):
        perm, _ = E.edl_shard_host(11, N, N, 1, epoch, 0)
        assert np.array_equal(np.sort(perm), np.arange(N))
        for t in sorted({0, 1, steps // 7, steps // 2, steps - steps // 50 - 1, steps - 2, steps - 1}):
            idx, _ = E.edl_shard_host(11, N, B, 1, epoch, t)
            assert np.array_equal(idx, perm[t * B:(t + 1) * B]), (epoch, t)


@pytest.mark.parametrize("N,B", [(1200000, 400), (401 * 2500, 401), (64 * 1563 + 8, 8), (2500000, 250)])
def test_shard_assignment_at_the_ends_of_the_sieve(E, N, B):
    """Steps sifted 64 at a time by the register tables and, from 401 entries on, by the table in memory; ends of the epoch that are
    no whole 64 steps."""
    test_shard_assignment_by_followed_entries(E, N, B)


def test_shard_errors(E):
    for args, code in [((0, 64, 8, 3, 0, 0), -2), ((0, 60, 8, 2, 0, 0), -2), ((0, 64, 8, 2, 0, 8), -4),
                       ((0, 64, 8, 0, 0, 0), -1), ((0, 64, 8, 2, -1, 0), -1)]:
        with pytest.raises(E.EdlError) as ei:
            E.edl_shard_host(*args)
        assert ei.value.code == code, args


ARCH_OF = {"resnet101": (64, 3, 4, 23, 3), "resnet152": (64, 3, 8, 36, 3), "vgg19": (64, 4096, 2, 2, 4, 4, 4)}


@pytest.mark.parametrize("model", ["mlp", "resnet20", "resnet50", "vgg16", "alexnet", "resnet101", "resnet152", "vgg19"])
def test_parameter_layout_and_init_match_the_oracle(E, model):
    from paper_1909_11985_amd.binding import make_config
    builder, kw = O.VARIANTS.get(model, (model, {}))
    cfg = make_config(builder, N=64, B=32, p_max=2, arch=ARCH_OF.get(model, ()))
    g = O.BUILDERS[builder](**kw)
    table = E.edl_tensor_table(cfg)
    assert table == [(n, o, int(np.prod(s)), f) for n, o, s, f in g.tensors]
    s = E.edl_query(cfg)
    assert (s.P, s.R) == (g.P, g.R)
    assert s.snapshot_bytes == O.SNAPSHOT_HEADER_BYTES + 4 * (2 * g.P + g.R)
    if model in ("mlp", "resnet20", "resnet50"):   # the larger ones (up to 144M Gaussians): covered on the GPU machine through the parity runs
        w = E.edl_init_params_host(cfg, 3)
        wo = O.he_init(g, 3)
        # both sides run Box-Muller in double and round to float32; allow a last-place difference of libm
        assert np.max(np.abs(w - wo)) <= 2.0 ** -23 * np.max(np.abs(wo))
        assert np.mean(w.astype(np.float64) != wo) < 1e-5


def test_adam_configuration_sizes_and_checks(E):
    from paper_1909_11985_amd.binding import make_config
    a = E.edl_query(make_config("resnet20", N=64, B=32, p_max=2))
    b = E.edl_query(make_config("resnet20", N=64, B=32, p_max=2, optimizer="adam"))
    assert a.second_off == -1 and b.second_off >= 0 and a.shadow_off == -1
    for s in (a, b, E.edl_query(make_config("resnet20", dtype="bf16", N=64, B=32, p_max=2, optimizer="adam"))):
        # the state arrays: disjoint, inside the arena, on 4 KB boundaries of alternating parity
        arrays = [(s.params_off, 4 * s.P), (s.momentum_off, 4 * s.P)]
        if s.second_off >= 0:
            arrays.append((s.second_off, 4 * s.P))
        if s.shadow_off >= 0:
            arrays.append((s.shadow_off, 2 * s.P))
        arrays += [(s.grads_off + 4 * s.grad_stride * k, 4 * s.P) for k in range(2)]
        arrays.append((s.running_off, 4 * s.R))
        spans = sorted(arrays)
        assert all(lo % 256 == 0 for lo, _ in spans) and spans[-1][0] + spans[-1][1] <= s.arena_bytes
        assert all(spans[i][0] + spans[i][1] <= spans[i + 1][0] for i in range(len(spans) - 1))
        pages = [lo for lo, _ in arrays[:-1]]
        assert all(lo % 4096 == 0 for lo in pages)
        assert (s.params_off >> 12) % 2 != (s.momentum_off >> 12) % 2             # w and v never on the same parity
        assert 4 * s.grad_stride % 8192 == 4096                                    # neighbouring gradient buffers neither
    assert b.snapshot_bytes == a.snapshot_bytes + 4 * a.P and b.arena_bytes >= a.arena_bytes + 4 * a.P
    for kw in [dict(momentum=1.0), dict(beta2=1.0), dict(beta2=-0.5), dict(eps=-1e-8), dict(optimizer=7)]:
        base = dict(model="mlp", N=64, B=32, p_max=2, optimizer="adam")
        base.update(kw)
        with pytest.raises(E.EdlError) as ei:
            E.edl_query(make_config(**base))
        assert ei.value.code == -1, kw
    E.edl_query(make_config("mlp", N=64, B=32, p_max=2, momentum=1.5))      # momentum-SGD does not restrict it


def test_query_rejects_bad_configurations(E):
    from paper_1909_11985_amd.binding import make_config
    for kw, code in [(dict(N=60, B=32), -2), (dict(p_max=17), -1), (dict(p_max=0), -1), (dict(model=9), -1), (dict(dtype=5), -1)]:
        base = dict(model="resnet50", N=64, B=32, p_max=2)
        base.update(kw)
        with pytest.raises(E.EdlError) as ei:
            E.edl_query(make_config(**base))
        assert ei.value.code == code, kw


def test_flops_per_sample(E):
    from paper_1909_11985_amd.binding import make_config
    # forward multiply-adds: 784*256 + 256*256 + 256*10; the first layer has no input gradient
    s = E.edl_query(make_config("mlp", N=64, B=32, p_max=2))
    assert s.flops_per_sample == 2 * (2 * 784 * 256 + 3 * 256 * 256 + 3 * 256 * 10)
    r = E.edl_query(make_config("resnet50", N=64, B=32, p_max=2))
    assert 23e9 < r.flops_per_sample < 25e9


# ---------------------------------------------------------------- dynamic data pipeline (host only)
@pytest.mark.parametrize("N,d,B", [(240, 12, 24), (240, 7, 24), (1000, 36, 40), (512, 512, 64), (360, 1, 12)])
def test_pipeline_matches_the_oracle_under_random_scaling(E, N, d, B):
    """Bit-exact against the oracle's leader over three epochs of joins and graceful exits."""
    import random
    from oracle.pipeline import DataPipeline
    rng = random.Random(N + 7 * d)
    lib_p, orc_p = E.Pipeline(11, N, d), DataPipeline(11, N, d)
    divisors = [p for p in range(1, B + 1) if B % p == 0 and p <= 12]
    workers = [0]
    for t in range(3 * (N // B)):
        if rng.random() < 0.6:
            p = rng.choice(divisors)
            keep = [w for w in workers if rng.random() < 0.6][:p]
            fresh = [w for w in range(50) if w not in workers]
            rng.shuffle(fresh)
            workers = keep + fresh[:p - len(keep)]
            rng.shuffle(workers)
        idx, off = lib_p.next_batch(B, workers)
        ref_idx, ref_off = orc_p.next_batch(B, workers)
        assert idx.tolist() == ref_idx and off.tolist() == ref_off, "mini-batch %d differs" % t
        assert lib_p.progress() == (orc_p.epoch, orc_p.consumed)
    lib_p.close()


def test_pipeline_at_the_sections_example_size(E):
    """1,000 partitions of 1,200 samples, 10 -> 15 -> 12 workers inside one epoch: same batches as the oracle."""
    from oracle.pipeline import DataPipeline
    N, d, B = 1_200_000, 1000, 600
    lib_p, orc_p = E.Pipeline(1, N, d), DataPipeline(1, N, d)
    steps = N // B
    for t in range(steps):
        workers = list(range(10)) if t < steps // 3 else list(range(15)) if t < steps // 2 else list(range(10)) + [10, 13]
        idx, off = lib_p.next_batch(B, workers)
        ref_idx, ref_off = orc_p.next_batch(B, workers)
        assert np.array_equal(idx, np.asarray(ref_idx)) and off.tolist() == ref_off
    assert lib_p.progress() == (0, N)


def test_pipeline_save_load_and_errors(E):
    a = E.Pipeline(8, 240, 16)
    sched = [[0, 1], [0, 1, 2], [2, 0], [5, 6, 7, 8], [5], [5, 9, 10], [1, 2]]
    for w in sched[:3]:
        a.next_batch(24, w)
    image = a.save()
    b = E.Pipeline.load(image)
    for w in sched[3:] * 3:
        ia, oa = a.next_batch(24, w)
        ib, ob = b.next_batch(24, w)
        assert np.array_equal(ia, ib) and np.array_equal(oa, ob)
    for bad in (image[:-1], np.concatenate([[7], image[1:]])):
        with pytest.raises(E.EdlError):
            E.Pipeline.load(bad)
    broken = image.copy()
    broken[7] = 10 ** 6                                       # cursor beyond d
    with pytest.raises(E.EdlError):
        E.Pipeline.load(broken)
    with pytest.raises(E.EdlError):
        E.Pipeline(0, 10, 11)
    with pytest.raises(E.EdlError):
        E.Pipeline(0, 10, 7)
    with pytest.raises(E.EdlError) as ei:
        a.next_batch(24, [3, 3])
    assert ei.value.code == -1
    with pytest.raises(E.EdlError) as ei:
        a.next_batch(24, [0, 1, 2, 3, 4])
    assert ei.value.code == -2
    with pytest.raises(E.EdlError) as ei:
        a.next_batch(36, [0, 1])                              # 36 does not divide 240
    assert ei.value.code == -2


def test_options_are_named_set_and_read_back(E):
    """The table of launch heuristics and code-path switches: defaults, a change and its undoing, unknown names."""
    assert E.edl_get_option("force_tile") == -1 and E.edl_get_option("wgrad_stream") == 1
    assert E.edl_get_option("early_update") == 16000000
    with E.options(force_tile=2, early_update=0):
        assert E.edl_get_option("force_tile") == 2 and E.edl_get_option("early_update") == 0
    assert E.edl_get_option("force_tile") == -1 and E.edl_get_option("early_update") == 16000000
    for bad in ("no_such_option", ""):
        with pytest.raises(E.EdlError) as ei:
            E.edl_set_option(bad, 1)
        assert ei.value.code == -1
        with pytest.raises(E.EdlError):
            E.edl_get_option(bad)


@pytest.mark.parametrize("model,dtype,kw", [("resnet20", "f32", {}), ("resnet20", "f32", dict(H=25, W=25)), ("resnet50", "bf16", {}),
                                            ("resnet50", "bf16", dict(H=161, W=161)), ("alexnet", "bf16", {}), ("vgg16", "f32", dict(H=64, W=64))])
def test_the_arena_holds_the_cut_weight_gradients_of_any_shards(E, model, dtype, kw):
    """A weight gradient is cut as its launch plans it, for the largest of a pass's shards: the arena has to hold the
    partial results for near-equal and for very unequal cuts, or the launch falls back to one cut per shard."""
    import random
    from paper_1909_11985_amd.binding import edl_debug_wgrad_scratch, make_config
    rng = random.Random(5)
    checked, cuts = 0, [[22, 21, 21], [17, 16, 16], [32, 32, 32, 32, 1], [64] + [1] * 7, [58, 2, 2, 2], [1], [7, 1], [1] * 16]
    for _ in range(60):
        p = rng.randint(1, 16)
        cuts.append([1 + int(rng.random() ** 3 * 36) for _ in range(p)])
    for cut in cuts:
        for max_shard in (max(cut), sum(cut)):
            cfg = make_config(model, dtype=dtype, N=sum(cut), B=sum(cut), p_max=len(cut), max_shard=max_shard, **kw)
            try:
                need, there = edl_debug_wgrad_scratch(cfg, cut)
            except E.EdlError as e:
                assert e.code == -4               # more than one pass: its parts are cuts like the others
                continue
            checked += 1
            assert need <= there, (cut, max_shard)
    assert checked > len(cuts)


@pytest.mark.parametrize("image,together", [(224, 4), (320, 2), (400, 1)])
def test_shards_run_together_only_as_far_as_the_vector_kernels_reach(E, image, together):
    """The convolution kernels' multiply-shift divisions are exact while samples * pixels^2 < 1e12: a pass of more
    shards than that would take the element-wise kernels where each shard alone takes the vector ones."""
    from paper_1909_11985_amd.binding import edl_debug_wgrad_scratch, make_config
    cfg = make_config("vgg16", dtype="bf16", N=128, B=128, p_max=4, max_shard=32, H=image, W=image, arch=(32, 64, 1, 1, 1, 1, 1))
    assert (32 * together * image ** 4 < 1e12) and (together == 4 or 32 * 4 * image ** 4 > 1e12)
    edl_debug_wgrad_scratch(cfg, [32] * together)
    if together < 4:
        with pytest.raises(E.EdlError) as ei:
            edl_debug_wgrad_scratch(cfg, [32] * 4)
        assert ei.value.code == -4


@pytest.mark.parametrize("model,dtype,kw", [("resnet50", "bf16", dict(B=256, p_max=8, max_shard=32)), ("resnet20", "f32", dict(B=128, p_max=8, max_shard=16)),
                                            ("vgg16", "bf16", dict(B=256, p_max=8, max_shard=32)), ("mlp", "f32", dict(B=64, p_max=4, max_shard=64))])
def test_a_job_can_be_held_to_the_memory_of_one_shard(E, model, dtype, kw):
    """The arena grows with the samples a pass may hold, from one shard's to what edl_query names; one shard's takes
    little more than the same job cut into mini-batches of that shard (its gradient buffers)."""
    from paper_1909_11985_amd.binding import make_config
    cfg = make_config(model, dtype=dtype, N=2 * kw["B"], **kw)
    full, least = E.edl_query(cfg), E.edl_arena_bytes(cfg)
    sizes = [E.edl_arena_bytes(cfg, n) for n in (1, kw["max_shard"], kw["B"] // 2, kw["B"], 10 * kw["B"])]
    assert least <= sizes[0] == sizes[1] <= sizes[2] <= sizes[3] <= sizes[4] == full.arena_bytes
    one = E.edl_query(make_config(model, dtype=dtype, N=kw["max_shard"], B=kw["max_shard"], p_max=1))
    assert least <= one.arena_bytes + 4 * (kw["p_max"] - 1) * full.grad_stride + 65536
    if kw["max_shard"] < kw["B"]:
        assert one.arena_bytes < full.arena_bytes / 2
    with pytest.raises(E.EdlError):
        E.edl_arena_bytes(cfg, -1)


@pytest.mark.parametrize("H,W,n,layers", [
    (1000, 1, 8000, 6), (1000, 1, 16770, 0), (1000, 1, 16800, 0),       # 2^24 rows of one pixel and more: the product has no room
    (4096, 1, 4100, 0), (2, 1, 5000, 16), (1000, 2, 8000, 6), (1000, 3, 8000, 6), (32, 32, 30000, 6),
])
def test_the_narrow_kernel_is_taken_only_where_its_divisions_are_exact(E, H, W, n, layers):
    """It numbers the pixels of a pass (up to 2^25) and divides those numbers by H W and by W with a product of 64 bits."""
    from paper_1909_11985_amd.binding import edl_debug_narrow_layers, make_config
    cfg = make_config("resnet20", N=n, B=n, p_max=1, max_shard=n, H=H, W=W)
    taken, M = edl_debug_narrow_layers(cfg, [n]), n * H * W
    assert taken == layers        # of 16 channels six, of 32 and 64 ten in all (not in passes of many blocks)
    numbers = sorted({x for c in (0, M // 2, 1 << 23, 1 << 24, M) for x in range(c - 130, c + 127) if 0 <= x < M + 127})
    exact = all(((x * (-(-(1 << 40) // d))) % (1 << 64)) >> 40 == x // d for x in numbers for d in (H * W, W))
    assert exact or taken == 0


# ---------------------------------------------------------------- device code
def _device_code(*flags, source="k_pointwise.hip"):
    """A source as the library is built of it, in text."""
    import subprocess
    from paper_1909_11985_amd import build
    cmd = ["hipcc", "-x", "hip", "-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", "-"] + build.FLAGS
    return subprocess.run(cmd + list(flags), check=True, capture_output=True, text=True).stdout


def test_streaming_kernels_order_their_lds_accesses():
    """A wave's outputs pass between its lanes through LDS behind a fence (before they are written, before they are read), and
    every barrier is reached with the wave's LDS writes done."""
    kernels = re.findall(r"^define [^\n]*pointwise_kernel[^\n]*\n(.*?)^}", _device_code("-emit-llvm"), flags=re.S | re.M)
    assert len(kernels) == 8
    for body in kernels:
        assert len(re.findall(r'fence syncscope\("wavefront"\) acq_rel', body)) >= 2
    code = [line.split(";")[0].strip() for line in _device_code().splitlines()]
    code = [line for line in code if line and not line.startswith(".")]
    barriers = [i for i, line in enumerate(code) if line == "s_barrier"]
    assert len(barriers) == 8
    for i in barriers:
        assert code[i - 1] == "s_waitcnt lgkmcnt(0)", code[i - 3:i + 1]


def test_streaming_kernels_keep_everything_in_registers():
    """Every variant that the dispatch reaches: registers in scratch cost a third of its speed."""
    code = _device_code()
    spills = dict(zip(re.findall(r"\.name: +(\S*pointwise_kernel\S*)", code), re.findall(r"\.vgpr_spill_count: +(\d+)", code)))
    assert len(spills) == 8 and set(spills.values()) == {"0"}, spills
    assert set(re.findall(r"\.private_segment_fixed_size: +(\d+)", code)) == {"0"}


def test_the_classifier_in_one_launch_orders_its_lds_accesses():
    """Logits and their gradients pass between the lanes of a wave through LDS: a fence before either is read."""
    kernels = re.findall(r"^define [^\n]*thin_head_kernel[^\n]*\n(.*?)^}", _device_code("-emit-llvm", source="k_thin.hip"), flags=re.S | re.M)
    assert len(kernels) == 2
    for body in kernels:
        assert len(re.findall(r'fence syncscope\("wavefront"\) acq_rel', body)) == 2
