"""Gradients of one training step at sizes where the training kernels' tiles
end unevenly: rows and columns that no stage divides (8-row and 16-column
stages at every level of the network, down to one row and one column at the
coarsest), several images, a partial last row, and enough pixels that the
weights-resident and persistent kernels run.  Reference: the oracle in
float64 over the images of the batch; tolerance per layer: twice the spread
of the oracle evaluated in float32 (+1 %), the bar of the other gradient
tests (a ReLU input or a max-pool pair within rounding distance of a tie
routes a whole gradient entry elsewhere in any two evaluations)."""
import numpy as np
import pytest

from test_gpu_learned import ctx, flat, fvv, rand_params, say, scene_stack, to_device_stack, unflat  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,W,valid", [(1, 8, 8, 8), (2, 8, 24, 7), (3, 24, 40, 21), (1, 72, 136, 72),
                                         (2, 136, 8, 130), (1, 264, 520, 260)])
def test_gradients_ragged(fvv, ctx, oracle_lib, N, H, W, valid):  # noqa: F811
    import torch
    from oracle import unet
    say(f"[gpu] gradients {N}x{H}x{W} valid={valid}")
    P = rand_params(400 + H + W)
    ctx.net_load(flat(P))
    st = np.stack([scene_stack(oracle_lib, 410 + q, W, H) for q in range(N)])
    target = np.random.default_rng(420).uniform(0, 1, (N, H, W, 3)).astype(np.float32)
    loss = ctx.net_train_step(to_device_stack(st), torch.from_numpy(target).cuda(), N, H, W, valid, lr=0.0,
                              apply=False)
    g = unflat(ctx.net_read(fvv.NET_GRADS))
    tot, ref, ref32 = 0.0, {}, {}
    for q in range(N):
        lq, rg = unet.loss_and_grads(P, st[q], target[q], valid)
        _, rg32 = unet.loss_and_grads(P, st[q], target[q], valid, acc=np.float32)
        tot += lq / N
        for name, *_ in unet.LAYERS:
            for k in (0, 1):
                ref[name, k] = ref.get((name, k), 0.0) + np.asarray(rg[name][k], np.float64).ravel() / N
                ref32[name, k] = ref32.get((name, k), 0.0) + np.asarray(rg32[name][k], np.float64).ravel() / N
    assert abs(loss - tot) <= 1e-3 * tot
    bad = []
    for (name, k), r in ref.items():
        nrm = max(np.linalg.norm(r), 1e-30)
        rel = np.linalg.norm(g[name][k].astype(np.float64).ravel() - r) / nrm
        floor = np.linalg.norm(ref32[name, k] - r) / nrm
        if rel > 2 * floor + 0.01:
            bad.append((name, "Wb"[k], rel, floor))
    assert not bad, bad


@pytest.mark.parametrize("N,H,W", [(17, 64, 264), (5, 232, 264)])
def test_batch_layers_equal_single(fvv, ctx, oracle_lib, N, H, W):  # noqa: F811
    """A batch large enough for the kernels of large grids (32-column patches
    at the half-resolution level, weights-resident ones at full resolution),
    whose images end their patches unevenly in rows and columns, gives every
    layer of its first and last image the bytes of that image alone, which
    runs in the kernels of small grids: each output's sum has the same order in
    all of them."""
    import torch
    from oracle import unet
    P = rand_params(500 + W)
    ctx.net_load(flat(P))
    st = to_device_stack(np.stack([scene_stack(oracle_lib, 510 + q % 2, W, H) for q in range(2)]))
    st = st[torch.arange(N, device="cuda") % 2].contiguous()
    level = dict(enc1a=1, enc1b=1, enc2a=2, enc2b=2, mid_a=3, mid_b=3, up2=2, dec2a=2, dec2b=2, up1=1, dec1a=1, dec1b=1)

    def layers(stack):
        n = stack.shape[0]
        out = torch.empty((n, H, W, 3), dtype=torch.float32, device="cuda")
        ctx.set_debug(True)
        ctx.net_forward(stack, n, H, W, out)
        torch.cuda.synchronize()
        ctx.set_debug(False)
        acts = {"out": out.cpu().numpy()}
        for i, (name, _, _, co) in enumerate(unet.LAYERS[:-1]):
            h, w = H >> level.get(name, 0), W >> level.get(name, 0)
            acts[name] = ctx.net_read_act(i, (n * h * w, co)).reshape(n, h, w, co)
        return acts

    many = layers(st)
    for q in (0, N - 1):
        one = layers(st[q:q + 1].contiguous())
        for name in one:
            assert np.array_equal(many[name][q], one[name][0]), (name, q)


@pytest.mark.parametrize("N,H,W", [(16, 136, 264), (64, 72, 104)])
def test_gradients_of_copies(fvv, ctx, oracle_lib, N, H, W):  # noqa: F811
    """The mean gradient over N copies of an image is the gradient of that
    image, which runs in the kernels of small grids; the copies run in those of
    large grids (strips and 32-column patches that end unevenly).  N is a power
    of two, so every gradient of the copies is the single one's scaled exactly
    and rounds to bfloat16 alike; only the order of the float32 sums over
    pixels differs: runs of at most 2^13 terms, relative rounding about
    2^-24 2^6.5, times 2^3 for what cancels within a layer: 1e-4."""
    import torch
    from oracle import unet
    say(f"[gpu] gradients of {N} copies {H}x{W}")
    ctx.net_load(flat(rand_params(430 + W)))
    st = scene_stack(oracle_lib, 431, W, H)
    target = np.random.default_rng(432).uniform(0, 1, (H, W, 3)).astype(np.float32)
    got = []
    for n in (1, N):
        ctx.net_train_step(to_device_stack(np.stack([st] * n)), torch.from_numpy(np.stack([target] * n)).cuda(), n, H, W,
                           H, lr=0.0, apply=False)
        got.append(unflat(ctx.net_read(fvv.NET_GRADS)))
    bad = []
    for name, *_ in unet.LAYERS:
        for k in (0, 1):
            a, b = (np.asarray(g[name][k], np.float64).ravel() for g in got)
            rel = np.linalg.norm(b - a) / max(np.linalg.norm(a), 1e-30)
            if not rel <= 1e-4:
                bad.append((name, "Wb"[k], rel))
    assert not bad, bad


@pytest.mark.parametrize("N,H,W", [(17, 64, 264), (5, 232, 264), (40, 72, 104), (72, 8, 480)])
def test_batch_output_equals_single(fvv, ctx, oracle_lib, N, H, W):  # noqa: F811
    """The same without debug taps: the batch computes the finest transposed
    convolution inside the next one and stores neither it nor the head's input;
    its strips end unevenly in rows and columns.  Bytes of the single image."""
    import torch
    ctx.net_load(flat(rand_params(520 + W)))
    st = to_device_stack(np.stack([scene_stack(oracle_lib, 530 + q, W, H) for q in range(2)]))
    st = st[torch.arange(N, device="cuda") % 2].contiguous()
    say(f"[gpu] outputs of {N} images {H}x{W}")

    def run(stack):
        out = torch.full((stack.shape[0], H, W, 3), 7.0, dtype=torch.float32, device="cuda")
        ctx.net_forward(stack, stack.shape[0], H, W, out)
        torch.cuda.synchronize()
        return out.cpu().numpy()

    many, one = run(st), [run(st[q:q + 1].contiguous())[0] for q in range(2)]
    for q in range(N):
        assert np.array_equal(many[q], one[q % 2]), q


@pytest.mark.parametrize("N,H,W,need", [(1, 8, 8, 2447872), (1, 64, 64, 7985664), (64, 8, 8, 7985664),
                                        (1, 128, 128, 27223296), (1, 256, 256, 108892416), (16, 64, 64, 108892416)])
def test_training_within_a_memory_budget(fvv, N, H, W, need):  # noqa: F811
    """A training step fits a context whose budget holds the weights and `need`
    bytes for the activation set (short of what the gradients' partial sums take
    where memory is free), and its gradients are those of a context without a
    budget up to the order of float32 sums: the norm of a sum of n terms in
    another order differs by less than sqrt(n) 2^-24 of the norm of the terms'
    magnitudes; 1e-5 of the gradient's norm allows for 64 K terms that cancel to
    a 40th."""
    import torch
    say(f"[gpu] training in a budget {N}x{H}x{W}")
    P = flat(rand_params(600 + H))
    g = torch.Generator(device="cuda").manual_seed(N + H)
    st = torch.rand((N, H, W, 16), generator=g, device="cuda").to(torch.bfloat16)
    st[..., 15] = 0
    target = torch.rand((N, H, W, 3), generator=g, device="cuda")

    def step(budget):
        c = fvv.Context(0, mem_budget=budget)
        c.net_load(P)
        weights = c.net_device_bytes()
        loss = c.net_train_step(st, target, N, H, W, H, lr=0.0, apply=False)
        grads, held = c.net_read(fvv.NET_GRADS), c.net_device_bytes()
        c.close()
        return loss, grads, weights, held

    loss, grads, weights, _ = step(0)
    loss_b, grads_b, _, held = step(weights + need)
    assert held <= weights + need and loss_b == loss
    a, b = unflat(grads), unflat(grads_b)
    for name in a:
        for k in (0, 1):
            d = np.linalg.norm(a[name][k].astype(np.float64) - b[name][k].astype(np.float64))
            assert d <= 1e-5 * np.linalg.norm(a[name][k].astype(np.float64)), (name, k)


@pytest.mark.parametrize("N,H,W", [(16, 520, 32), (64, 264, 16), (64, 520, 8)])
def test_narrow_batches(fvv, ctx, oracle_lib, N, H, W):  # noqa: F811
    """Batches of images no wider than 16 pixels at the levels with 64 K pixels
    and more, which take patches of 16 columns (16, 8 and 4 columns, rows
    that end patches unevenly), and no wider than 8 at the finest, where the
    finest transposed convolution stays a launch of its own: layers and outputs
    have the bytes of the single image."""
    say(f"[gpu] narrow batch {N}x{H}x{W}")
    test_batch_layers_equal_single(fvv, ctx, oracle_lib, N, H, W)
    test_batch_output_equals_single(fvv, ctx, oracle_lib, N, H, W)
