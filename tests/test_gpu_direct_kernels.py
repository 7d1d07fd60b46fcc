"""The register-fed kernels at the edges of their tiles and dispatch rules,
against the oracle on the same seeded inputs.

* MLP: the fused head at 16, 17, 33, 64 classes and the separate path at 65;
  batches of one row, around 16 and past 128; widths and K that leave ragged
  32-wide K tiles and ragged output tiles; the 64 x 64 update tiles with a
  gathered first layer whose batch is no multiple of 16.
* The fused bf16 head: 32, 33 and 64 classes (65: the separate launches), one
  K chunk, a ragged second one, and more chunks than the waves take at once.
* Convolutions: a gathered first layer on the direct kernels (4 and 16
  channels), K groups within one tap (channels a multiple of 16) and across taps
  (4, 12, 20), 1 to 3 output-channel blocks, stride 2 on odd sizes, several
  pixel ranges with a ragged last one, pixels beyond one tile of every kind
  (16-channel layers by 64 pixels with many replicas), images of more than 2^20
  pixels, the tallest ones, weights that keep the ranges long; and the general
  kernels' 16-byte loads where one side's channels are in fours.
* Evaluation over several passes with a ragged last one, MLP (fp32 and bf16, with
  buffers of its own and without, the softmax in the head and apart) and CNN.

The tolerance is FP32_TOL (BF16_TOL) of the trajectory tests: these are sums of the same
lengths (K up to 2304, pixels up to 4800) in fp32, whose order alone differs."""
import numpy as np
import pytest

import oracle
import workload
from _parity import BF16_TOL, FP32_TOL, assert_tensors_close, gpu_rounds, oracle_rounds, say, tensor_errors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2102_08550_amd
    return paper_2102_08550_amd


def _mlp(dims, batch, tau, seed, dtype=workload.FP32):
    return workload.Config("direct-mlp", dims, dtype, K=len(tau), n_rows=4 * batch + 3,
                           batch=batch, tau_rule="given", tau_given=tau, lr=0.05, rounds=1,
                           seed=seed)


def _cnn(image, conv, batch, tau, seed, classes=10):
    return workload.Config("direct-cnn", (image[0] * image[1] * image[2], classes), workload.FP32,
                           K=len(tau), n_rows=4 * batch + 3, batch=batch, tau_rule="given",
                           tau_given=tau, lr=0.1, rounds=1, seed=seed, image=image, conv=conv,
                           mean_scale=0.5)


CASES = {
    "head-16": _mlp((24, 40, 16), 15, (2, 1), 101),
    "head-17": _mlp((40, 72, 17), 16, (2, 1), 102),
    "head-33": _mlp((136, 264, 33), 17, (1, 2), 103),
    "head-64": _mlp((264, 1032, 64), 1, (2, 3), 104),
    "classes-65": _mlp((72, 104, 65), 33, (2, 1), 105),
    "softmax": _mlp((792, 10), 65, (3, 0, 2), 106),
    "update-64": _mlp((1032, 2056, 10), 130, (1, 2, 1), 107),
    "update-pairs": _mlp((1032, 2056, 10), 130, (1,) * 7, 109),
    "update-alone": _mlp((1032, 2056, 10), 200, (1, 1, 1), 110),
    "update-last": _mlp((2056, 1544, 136), 128, (2,), 108),
    "bf16-head-32": _mlp((16, 24, 32), 1, (2, 1), 131, workload.BF16),
    "bf16-head-33": _mlp((40, 1032, 33), 33, (2, 1), 132, workload.BF16),
    "bf16-head-64": _mlp((24, 9224, 64), 31, (1, 2), 133, workload.BF16),
    "bf16-classes-65": _mlp((72, 2056, 65), 40, (2, 1), 134, workload.BF16),
    "gather-4": _cnn((9, 11, 4), ((4, 1), (12, 2)), 5, (2, 1), 111),
    "gather-16": _cnn((8, 6, 16), ((16, 1), (32, 1)), 6, (2, 1), 112),
    "taps-cross": _cnn((7, 9, 3), ((20, 1), (12, 1), (36, 2)), 7, (1, 2), 113),
    "blocks-3": _cnn((11, 13, 3), ((48, 1), (68, 2), (68, 1), (68, 1, 1)), 4, (2, 1), 114),
    "ranges": _cnn((20, 20, 3), ((16, 1), (32, 1), (64, 2)), 12, (1, 2), 115),
    "ranges-wide": _cnn((8, 8, 3), ((384, 1), (392, 1), (384, 2)), 9, (1, 2), 118),
    "image-1030x1020": _cnn((1030, 1020, 4), ((4, 1), (8, 2)), 1, (1,), 117),
    "image-4096x2": _cnn((4096, 2, 4), ((12, 1), (16, 2), (16, 1)), 2, (1, 2), 119),
    "fours-on-one-side": _cnn((11, 9, 4), ((10, 1), (12, 2), (7, 1), (8, 2), (6, 1)), 5, (2, 1), 122),
    "tiles-16x64": _cnn((32, 32, 3), ((16, 1), (16, 1), (32, 2)), 128, (1,) * 8, 120),
    "many-slots": _cnn((16, 16, 3), ((32, 1), (64, 2), (64, 1, 0)), 16, (1, 1, 1, 1, 1), 116),
}


@pytest.mark.parametrize("name", CASES)
def test_direct_kernels_match_oracle(P, name):
    cfg = CASES[name]
    say(f"direct {name}: dims={cfg.dims} image={cfg.image} conv={cfg.conv} B={cfg.batch}")
    ds = workload.gen_dataset(cfg)
    init = workload.gen_init(cfg)
    tau = np.array([cfg.tau_given])
    g_gpu, l_gpu = gpu_rounds(cfg, ds, init, tau, fused=False)
    g_ref, l_ref = oracle_rounds(cfg, ds, init, tau)
    tol = BF16_TOL if cfg.dtype == workload.BF16 else FP32_TOL
    assert_tensors_close(tensor_errors(g_gpu[0], g_ref[0]), tol, name)
    for k in range(cfg.K):
        if tau[0][k]:
            assert abs(l_gpu[0][k] - l_ref[0][k]) <= tol * max(abs(l_ref[0][k]), 1e-2), k


# One row, one pass less one row, exactly one, and one with a ragged second.
@pytest.mark.parametrize("rows", [1, 8191, 8192, 8192 + 70])
def test_evaluation_passes_match_oracle(P, rows):
    import torch
    cfg = _mlp((40, 72, 17), 16, (1, 1), 121)
    say(f"evaluate {rows} rows")
    init = workload.gen_init(cfg)
    ctx = P.Context(cfg.dims, P.FP32, cfg.K, cfg.batch)
    try:
        ev = workload.gen_eval_set(cfg, rows)
        loss, hits = ctx.evaluate(torch.from_numpy(ctx.pack(init)).cuda(),
                                  torch.from_numpy(ev.x).cuda(),
                                  torch.from_numpy(ev.y.astype(np.int32)).cuda())
        ref_loss, ref_hits, gaps = oracle.mlp.evaluate(
            [(W.astype(np.float64), b.astype(np.float64)) for W, b in init],
            ev.x.astype(np.float64), ev.y)
        assert abs(loss - ref_loss) <= FP32_TOL * abs(ref_loss)
        assert abs(hits - ref_hits) <= int((np.asarray(gaps) < 1e-4).sum())  # rounding decides these
    finally:
        ctx.close()


# Several passes: bf16 rows (two passes of 8192 and a ragged third), more
# activations of the local steps than a pass of its own would have (their rows
# are the pass), the softmax apart (65 classes and more), and convolutions (K x
# max_batch images per pass, in slots of one or several rows).
EVALUATIONS = {
    "bf16": (_mlp((40, 72, 48, 17), 16, (1, 1), 171, workload.BF16), [8192, 2 * 8192 + 70]),
    "bf16-classes-130": (_mlp((264, 136, 130), 16, (1, 1), 172, workload.BF16), [8192 + 1]),
    "own-rows": (_mlp((24, 40, 17), 1024, (1,) * 9, 173), [9216, 9216 + 70]),
    "own-rows-bf16": (_mlp((24, 40, 72), 1024, (1,) * 9, 174, workload.BF16), [9216 + 70]),
    "classes-65": (_mlp((40, 72, 65), 16, (1, 1), 175), [8191, 8192 + 70]),
    "one-layer-100": (_mlp((40, 100), 16, (1, 1), 176), [8192 + 70]),
    "one-layer-head": (_mlp((40, 10), 16, (1, 1), 178), [8192 + 70]),
    "cnn": (_cnn((9, 7, 3), ((8, 1), (12, 2)), 16, (1, 1, 1), 177), [1, 47, 48, 49, 130]),
}


@pytest.mark.parametrize("name", EVALUATIONS)
def test_evaluation_paths_match_oracle(P, name):
    import torch
    cfg, sizes = EVALUATIONS[name]
    say(f"evaluate {name}")
    init = workload.gen_init(cfg)
    bf16 = cfg.dtype == workload.BF16
    ref = [(W.astype(np.float64), b.astype(np.float64)) for W, b in init]
    cnn = (cfg.image, cfg.conv) if cfg.image else None
    ctx = P.Context(cfg.dims, P.BF16 if bf16 else P.FP32, cfg.K, cfg.batch, cnn=cnn)
    try:
        flat = torch.from_numpy(ctx.pack(init)).cuda()
        for rows in sizes:
            ev = workload.gen_eval_set(cfg, rows)
            x = torch.from_numpy(np.ascontiguousarray(ev.x.view(np.int16) if bf16 else ev.x)).cuda()
            y = torch.from_numpy(ev.y.astype(np.int32)).cuda()
            loss, hits = ctx.evaluate(flat, x, y)
            assert ctx.evaluate(flat, x, y, noalloc=True) == (loss, hits)
            x64 = ev.x_f32().astype(np.float64)
            if cnn:
                ref_loss, ref_hits = oracle.cnn.evaluate(ref, x64, ev.y, cfg.image, cfg.strides,
                                                         cfg.skips)
                near = 1
            else:
                ref_loss, ref_hits, gap = oracle.mlp.evaluate(ref, x64, ev.y, bf16)
                near = int((gap < (1e-2 if bf16 else 1e-4)).sum())  # rounding decides these
            assert abs(loss - ref_loss) <= (BF16_TOL if bf16 else FP32_TOL) * abs(ref_loss), rows
            assert abs(hits - ref_hits) <= near, rows
    finally:
        ctx.close()


def test_context_without_room_for_evaluation_buffers(P):
    """A context is created where the 64 MiB for wide evaluation passes no
    longer fit, and evaluates in passes of its local steps' rows."""
    import torch
    say("evaluation without buffers of its own")
    cfg = _mlp((16, 1024, 17), 16, (1, 1), 151)
    init = workload.gen_init(cfg)
    ev = workload.gen_eval_set(cfg, 100)
    args = (torch.from_numpy(ev.x).cuda(), torch.from_numpy(ev.y.astype(np.int32)).cuda())
    ctx = P.Context(cfg.dims, P.FP32, cfg.K, cfg.batch)
    flat = torch.from_numpy(ctx.pack(init)).cuda()
    ref = ctx.evaluate(flat, *args)
    ctx.close()
    ballast = []
    for size in (1 << 32, 1 << 28, 1 << 24):  # until not even 16 MiB are free
        try:
            while True:
                ballast.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            pass
    del ballast[-2:]  # 32 MiB for the rest of the context
    torch.cuda.empty_cache()
    try:
        ctx = P.Context(cfg.dims, P.FP32, cfg.K, cfg.batch)
    finally:
        del ballast
        torch.cuda.empty_cache()
    try:
        assert ctx.evaluate(flat, *args) == ref
    finally:
        ctx.close()


def test_weight_gradient_partials_fit_the_pixels(P):
    """A context holds the partials of the ranges that its batches have, not of
    a fixed number: one copy of the weights for 128 pixels, and a batch of fewer
    pixels than max_batch's may have more ranges (63 against 64 images here)."""
    import torch
    say("weight-gradient partials")
    image, conv = (4, 4, 8), ((1024, 1), (1024, 1))
    K, batch = 2, 8
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx = P.Context((128, 10), P.FP32, K, batch, cnn=(image, conv))
    try:
        used = free - torch.cuda.mem_get_info()[0]
        partials = K * 4 * ctx.n_pad
        activations = K * batch * 16 * 2 * 2 * 1024 * 4
        assert used <= partials + activations + (64 << 20), (used, partials, activations)
    finally:
        ctx.close()
    cfg = _cnn((8, 8, 4), ((16, 1), (32, 1)), 63, (2, 1), 152)
    ds, init = workload.gen_dataset(cfg), workload.gen_init(cfg)
    x, y = torch.from_numpy(ds.x).cuda(), torch.from_numpy(ds.y.astype(np.int32)).cuda()
    out = []
    for max_batch in (63, 64):
        ctx = P.Context((256, 10), P.FP32, cfg.K, max_batch, cnn=(cfg.image, cfg.conv))
        try:
            flat = torch.from_numpy(np.tile(ctx.pack(init), cfg.K)).cuda()
            ctx.local_steps(flat, x, y, P.shard_offsets(cfg.n_rows, cfg.K), 5, cfg.tau_given, 0.1, 63)
            out.append(flat.cpu())
        finally:
            ctx.close()
    assert torch.equal(out[0].view(torch.int32), out[1].view(torch.int32))


def test_large_images_take_the_paired_backward(P):
    """Layers whose channel counts are multiples of 4 run backward-data and
    backward-weight in one launch whatever the size of their images."""
    import torch
    image, conv = (1030, 1020, 4), ((4, 1), (8, 2))
    say(f"paired backward, image {image}")
    d = image[0] * image[1] * image[2]
    ctx = P.Context((d, 10), P.FP32, 1, 1, cnn=(image, conv))
    try:
        flat = torch.zeros(ctx.n_pad).cuda()
        ctx.profile_begin(range(len(P.KERNEL_NAMES)))
        ctx.local_steps(flat, torch.ones((2, d)).cuda(), torch.zeros(2, dtype=torch.int32).cuda(),
                        [0, 2], 1, [1], 0.1, 1)
        launches = {k: n for k, (_, n) in ctx.profile_end().items()}
        assert launches["gemm_bwd_fused"] == 1, launches  # layer 2
    finally:
        ctx.close()


WIDE = 65536  # the widest accepted layer
BIG = 2.0 ** 27
# A product of 2^27 followed by ones: a running sum that has reached 2^27 (ulp 16)
# loses every one that it adds.  Runs of at most 1024 products lose 1023 of
# them; every other run is a whole number below 2^24, and adding it to the
# total rounds by at most 8.  At most 64 + 8 such additions.  (A slice of 16384
# or 8192 in one run loses all of its ones.)
WIDE_BOUND = 1023 + (64 + 8) * 8


def _context(P, torch, dims):
    ctx = P.Context(dims, P.FP32, 1, 1)
    y = torch.tensor([dims[-1] - 1], dtype=torch.int32).cuda()  # the last class
    return ctx, y


def _weights(dims):
    return [(np.zeros((o, i), np.float32), np.zeros(o, np.float32))
            for i, o in zip(dims, dims[1:])]


def _step(ctx, torch, layers, x, y, lr):
    flat = torch.from_numpy(ctx.pack(layers)).cuda()
    ctx.local_steps(flat, x, y, [0, 1], 1, [1], lr, 1)
    return ctx.unpack(flat.cpu().numpy())


@pytest.mark.parametrize("tiling", ["L", "M", "S"])
def test_wide_layers_sum_in_runs_of_1024(P, tiling):
    """Forward (gathered and not) and backward-data of a layer of 65536 inputs
    (outputs), whose values are read off one update or the loss exactly: all
    factors around them are powers of two."""
    import torch
    say(f"wide sums, tiling {tiling}")
    lr = 2.0 ** -20
    dims = (WIDE, 8, 2)
    ctx, y = _context(P, torch, dims)
    try:
        ctx.set_gemm_tiling(P.TILINGS[tiling])
        layers = _weights(dims)
        layers[0][0][3] = 1.0
        layers[0][0][3, 0] = BIG
        x = torch.ones((1, WIDE)).cuda()
        true = BIG + WIDE - 1
        # zero W_2: delta_2 = (1/2, -1/2), W_2 <- 0 - lr delta_2 a_1
        a1 = float(_step(ctx, torch, layers, x, y, lr)[1][0][1, 3]) / (lr * 0.5)
        assert abs(a1 - true) <= WIDE_BOUND, a1 - true
        # logits (a_1, 0), label 1: the loss is a_1
        layers[1][0][0, 3] = 1.0
        loss, _ = ctx.evaluate(torch.from_numpy(ctx.pack(layers)).cuda(), x, y)
        assert abs(loss - true) <= WIDE_BOUND, loss - true
    finally:
        ctx.close()
    dims = (8, 8, WIDE)
    ctx, y = _context(P, torch, dims)
    try:
        ctx.set_gemm_tiling(P.TILINGS[tiling])
        # logits of at most 2^-33: the softmax is uniform, delta_2 = 2^-16 but
        # for the label, whose weight is zero
        layers = _weights(dims)
        layers[0][1][5] = 2.0 ** -60
        layers[1][0][:, 5] = 1.0
        layers[1][0][0, 5] = BIG
        layers[1][0][WIDE - 1, 5] = 0.0
        x = torch.zeros((1, 8)).cuda()
        x[0, 2] = 1.0
        d1 = float(_step(ctx, torch, layers, x, y, lr)[0][0][5, 2]) / (-lr * 2.0 ** -16)
        assert abs(d1 - (BIG + WIDE - 2)) <= WIDE_BOUND, d1 - (BIG + WIDE - 2)
    finally:
        ctx.close()


@pytest.mark.parametrize("classes", [2, 17, 33])
def test_wide_head_sums_in_runs_of_1024(P, classes):
    """The fused head on 65536 inputs, its rows gathered (local steps), and
    not (evaluation, and below a hidden layer)."""
    import torch
    say(f"wide head, {classes} classes")
    true = BIG + WIDE - 1
    dims = (WIDE, classes)
    ctx, y = _context(P, torch, dims)
    try:
        layers = _weights(dims)
        layers[0][0][0] = 1.0
        layers[0][0][0, 0] = BIG
        x = torch.ones((1, WIDE)).cuda()
        flat = torch.from_numpy(ctx.pack(layers)).cuda()
        loss, _ = ctx.evaluate(flat, x, y)  # the largest logit is all of the loss
        assert abs(loss - true) <= WIDE_BOUND, loss - true
        ctx.local_steps(flat, x, y, [0, 1], 1, [1], 2.0 ** -20, 1)
        loss = float(ctx.round_losses()[0])
        assert abs(loss - true) <= WIDE_BOUND, loss - true
    finally:
        ctx.close()
    dims = (8, WIDE, classes)
    ctx, y = _context(P, torch, dims)
    try:
        layers = _weights(dims)
        layers[0][1][:] = 1.0  # activations of one
        layers[1][0][0] = 1.0
        layers[1][0][0, 0] = BIG
        _step(ctx, torch, layers, torch.zeros((1, 8)).cuda(), y, 2.0 ** -20)
        loss = float(ctx.round_losses()[0])
        assert abs(loss - true) <= WIDE_BOUND, loss - true
    finally:
        ctx.close()


@pytest.mark.parametrize("dims,one_launch", [((24, 4096, 64), True), ((24, 4104, 64), False),
                                             ((24, 8192, 10), True), ((24, 8200, 10), False)])
def test_bf16_head_or_split_k_by_depth(P, dims, one_launch):
    """With split-K partials in the context (batches above 128) a last layer
    deeper than the head's one turn of K chunks takes the separate launches;
    without, the head.  The same bits either way."""
    import torch
    say(f"bf16 head {dims}")
    cfg = _mlp(dims, 40, (2, 1), 141, workload.BF16)
    ds, init = workload.gen_dataset(cfg), workload.gen_init(cfg)
    x = torch.from_numpy(np.ascontiguousarray(ds.x).view(np.int16)).cuda()
    y = torch.from_numpy(ds.y.astype(np.int32)).cuda()
    out = []
    for max_batch in (cfg.batch, 256):
        ctx = P.Context(cfg.dims, P.BF16, cfg.K, max_batch)
        try:
            flat = torch.from_numpy(np.tile(ctx.pack(init), cfg.K)).cuda()
            ctx.profile_begin(range(len(P.KERNEL_NAMES)))
            ctx.local_steps(flat, x, y, P.shard_offsets(cfg.n_rows, cfg.K), 5, cfg.tau_given, 0.05,
                            cfg.batch)
            launches = {k: n for k, (_, n) in ctx.profile_end().items()}
            # two local steps: layer 1, and the last layer where it is not in the head
            head = max_batch == cfg.batch or one_launch
            assert launches["gemm_fwd"] == (2 if head else 4), launches
            assert launches["softmax_ce"] == 2
            out.append((flat.cpu().numpy(), ctx.round_losses()))
        finally:
            ctx.close()
    assert np.array_equal(out[0][0].view(np.uint32), out[1][0].view(np.uint32))
    assert np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("batch", [130, 200])
def test_update_tiles_give_the_same_bits(P, batch):
    """Seven replicas take 64 x 64 update tiles, two waves per SIMD (batch 130) or
    one (200), a single one 32 x 32 tiles: a replica's bits are the same."""
    import torch
    say(f"update tiles, batch {batch}")
    cfg = _mlp((1032, 2056, 10), batch, (1,) * 7, 142)
    ds, init = workload.gen_dataset(cfg), workload.gen_init(cfg)
    x, y = torch.from_numpy(ds.x).cuda(), torch.from_numpy(ds.y.astype(np.int32)).cuda()
    off = P.shard_offsets(cfg.n_rows, cfg.K)
    ctx = P.Context(cfg.dims, P.FP32, cfg.K, batch)
    try:
        start = torch.from_numpy(np.tile(ctx.pack(init), cfg.K)).cuda()
        flat = start.clone()
        ctx.local_steps(flat, x, y, off, 5, [1] * 7, 0.05, batch)
        for k in (0, 6):
            solo = start.clone()
            ctx.set_cursors([0] * 7)
            ctx.local_steps(solo, x, y, off, 5, [int(j == k) for j in range(7)], 0.05, batch)
            n = ctx.n_pad
            assert torch.equal(solo[k * n:(k + 1) * n].view(torch.int32),
                               flat[k * n:(k + 1) * n].view(torch.int32)), k
    finally:
        ctx.close()


@pytest.mark.parametrize("dims,dtype,batch", [
    ((24, 10), "fp32", 9), ((24, 40, 10), "fp32", 9), ((24, 40, 32, 65), "fp32", 9),
    ((24, 10), "bf16", 9), ((24, 40, 32, 10), "bf16", 9), ((24, 4104, 64), "bf16", 130)])
def test_bench_books_work_on_the_launches_that_run(P, dims, dtype, batch):
    """Kinds of launches with products in the benchmark's count are the kinds
    that a round launches."""
    import torch

    import bench
    cfg = _mlp(dims, batch, (1, 2), 161, getattr(workload, dtype.upper()))
    say(f"booked work {dims} {dtype}")
    ds, init = workload.gen_dataset(cfg), workload.gen_init(cfg)
    x = ds.x.view(np.int16) if dtype == "bf16" else ds.x
    ctx = P.Context(cfg.dims, getattr(P, dtype.upper()), cfg.K, batch)
    try:
        ctx.set_backward(P.BACKWARDS["separate"])
        flat = torch.from_numpy(np.tile(ctx.pack(init), cfg.K)).cuda()
        ctx.profile_begin(range(len(P.KERNEL_NAMES)))
        ctx.local_steps(flat, torch.from_numpy(np.ascontiguousarray(x)).cuda(),
                        torch.from_numpy(ds.y.astype(np.int32)).cuda(),
                        P.shard_offsets(cfg.n_rows, cfg.K), 5, cfg.tau_given, 0.05, batch)
        launches = {k: n for k, (_, n) in ctx.profile_end().items()}
        work = bench.gemm_work(cfg, cfg.tau_given, lambda l, ns: False)
        for kind in ("gemm_fwd", "gemm_dgrad", "gemm_wgrad_update", "gemm_bwd_fused"):
            assert (work[kind][0] > 0) == (launches[kind] > 0), (kind, launches)
    finally:
        ctx.close()
