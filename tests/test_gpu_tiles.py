"""The fp32 spatial tiles at the edges of their boxes (widths that leave part
of a box empty, boxes over the end of an image, one image, rows longer than a
box, channel counts in fours), the stem kernels, the stride-2 data gradient on
odd grids, pooled heads over large maps, the 2x2 max-pool gradient, weight
gradients over many boxes and channel blocks, infinities, tensors over 2 GiB,
the bf16 ReLU decision recomputed, and the threaded copies to the host:
against the fp64 oracle with the bars of tests/parity.py, or bit for bit where
nothing is rounded."""
import sys
import threading

import numpy as np
import pytest

import synth
from oracle import lppref as R
from oracle import models as OM
from paper_2203_06638_amd import lpp
from paper_2203_06638_amd import models as PM
from tests import parity as T

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _device():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    torch.cuda.init()


def dev(img, lab):
    return (torch.from_numpy(np.ascontiguousarray(img)).cuda(),
            torch.from_numpy(np.ascontiguousarray(lab, np.int32)).cuda())


def grid_inputs(o, seed, n):
    """Images and first-conv weights on exact grids: the first conv's output,
    which the ReLU or the pool decides on, is exact in both precisions."""
    x = T.init_x(o.specs, seed)
    rec = o.layers[0]
    nw = rec["cout"] * rec["cin"] * rec["k"] ** 2
    x[:nw] = synth.grid_values(seed, nw, 2.0 ** -5, 0.5)
    return x, synth.grid_values(seed + 1, (n,) + o.in_shape, 2.0 ** -6, 4.0), synth.labels(seed, n, o.n_classes)


def check_step(o, p, n, seed=11, modes=(lpp.SEQUENTIAL, lpp.ASYNC)):
    x, img, lab = grid_inputs(o, seed, n)
    loss, logits, _ = R.forward_backward(o, x, img, lab)
    g, sc = R.grad_scale(o, x, img, lab)
    for mode in modes:
        with lpp.Context(p, K=1, batch=n, mode=mode) as ctx:
            ctx.set_params(x)
            i, t = dev(img, lab)
            torch.cuda.synchronize()
            ctx.step(0, i, t, 0, 0.0)
            assert T.relerr(ctx.get_logits(0), logits, T.TAU_LOGITS) < T.TOL_LOGITS
            worst = T.worst(T.tensor_errors(o, ctx.get_grad(0), g, scale=sc))
            print(o.in_shape, n, "mode", mode, "worst", worst, file=sys.stderr, flush=True)
            assert worst[1] < T.TOL_GRAD, worst


# cin, c1, k, stride, pad, c2, hw, batch: image -> conv -> ReLU -> conv 3x3 -> pool -> linear
@pytest.mark.parametrize("case", [
    (3, 16, 3, 1, 1, 16, 7, 1),       # one image smaller than a box
    (3, 20, 3, 1, 1, 36, 28, 5),      # channels in fours, boxes over the images' ends
    (3, 24, 3, 2, 1, 16, 33, 3),      # stem of stride 2, odd size
    (3, 64, 7, 2, 3, 20, 47, 2),      # 7x7/2 stem, ragged output channels
    (3, 32, 7, 1, 3, 16, 11, 3),      # 7x7 stem of stride 1
    (4, 16, 3, 1, 1, 16, 130, 1),     # rows longer than a box, four image channels
    (3, 16, 3, 1, 1, 64, 20, 3),      # head over 20x20x64: pool and broadcast passes of their own
    (3, 16, 3, 1, 0, 16, 30, 2),      # unpadded stem
    (3, 48, 3, 1, 1, 52, 14, 9),
], ids=lambda c: "x".join(map(str, c)))
def test_tile_edges(case):
    cin, c1, k, st, pad, c2, hw, n = case
    check_step(*T.twin_conv_net(cin, c1, k, st, pad, c2, hw), n)


# cin, c0, c1, k, stride, pad, hw, batch: image -> conv 3x3 -> ReLU -> conv -> pool -> linear
@pytest.mark.parametrize("case", [
    (3, 16, 36, 3, 2, 1, 17, 3),      # parity-split data gradient, odd grid
    (3, 20, 24, 1, 2, 0, 15, 4),
    (3, 16, 16, 3, 2, 1, 28, 37),     # several boxes a workgroup
    (3, 32, 32, 1, 1, 0, 9, 5),
    (3, 32, 64, 1, 1, 0, 40, 12),     # 32-channel 1x1 tiles
    (3, 16, 32, 3, 3, 1, 19, 3),      # stride 3: the gather data gradient
    (3, 320, 320, 3, 1, 1, 10, 3),    # weight gradient of 400 channel blocks
    (3, 128, 256, 3, 2, 1, 9, 2),     # stride 2 of many blocks, few pixels
    (3, 128, 256, 3, 2, 1, 33, 15),   # weight gradients on the GEMM kernel: more pixels,
    (3, 64, 80, 1, 1, 0, 60, 20),     # large 1x1 passes,
    (3, 64, 64, 1, 1, 0, 32, 64),     # rows of 2^k
    (3, 32, 64, 1, 1, 0, 32, 40),     # 1x1 weight gradients of single full boxes,
    (3, 32, 64, 1, 1, 0, 32, 80),     # and of runs
], ids=lambda c: "x".join(map(str, c)))
def test_second_conv_edges(case):
    cin, c0, c1, k, st, pad, hw, n = case
    check_step(*T.twin_conv2_net(cin, c0, c1, k, st, pad, hw), n)


@pytest.mark.parametrize("hw,n,widths", [(13, 5, (16, 20, 32)), (22, 3, (20, 36, 16))])
def test_folded_batch_norm_on_ragged_boxes(hw, n, widths):
    """ResNet units whose BN + ReLU folds and backward sums run on ragged
    boxes: statistics by counted tiles, folded staging, sums in the data
    gradient's epilogue.  BN shifts +4 and -4 on alternate channels keep every
    ReLU decision clear of both precisions' disagreement."""
    o, p = OM.resnet_cifar(1, widths, 10, hw), PM.resnet_cifar(8, widths, 10, hw)
    o.set_blocks([1] * 5)

    def make(seed):
        x = T.init_x(o.specs, seed)
        for name, off, cnt in o.tensors:
            if name.endswith("bn_beta"):
                x[off:off + cnt] = np.where(np.arange(cnt) % 2 == 0, 4.0, -4.0)
        return x.astype(np.float64), T.inputs(seed + 7, n, o.in_shape, 10)[0]

    seed, _ = T.well_posed_seed(o, make, seeds=range(2600, 2680), band=1e-5)
    x = make(seed)[0].astype(np.float32)
    img, lab = T.inputs(seed + 7, n, o.in_shape, 10)
    _, logits, _ = R.forward_backward(o, x, img, lab)
    g, sc = R.grad_scale(o, x, img, lab)
    for mode in (lpp.SEQUENTIAL, lpp.ASYNC):
        with lpp.Context(p, K=1, batch=n, mode=mode) as ctx:
            ctx.set_params(x)
            i, t = dev(img, lab)
            torch.cuda.synchronize()
            ctx.step(0, i, t, 0, 0.0)
            assert T.relerr(ctx.get_logits(0), logits, T.TAU_LOGITS) < T.TOL_LOGITS
            worst = T.worst(T.tensor_errors(o, ctx.get_grad(0), g, scale=sc))
            print("hw", hw, "mode", mode, "worst", worst, file=sys.stderr, flush=True)
            assert worst[1] < T.TOL_GRAD, worst


@pytest.mark.parametrize("hw", [13, 14])
def test_maxpool_gradient_blocks(hw):
    """conv -> max pool 3x3/2 padded by 1 -> conv on odd and even maps: the
    argmax decisions are taken on identical values (exact grid)."""
    o = OM.Net("poolnet", 3, hw, hw, 6)
    a = o.maxpool(o.conv(-1, 3, 16, 3, 1, 1), 3, 2, 1)
    a = o.gap(o.conv(a, 16, 16, 3, 1, 1))
    o.next_unit()
    o.linear(a, 16, 6)
    o.set_blocks([1, 2])
    p = PM.Model("poolnet", (3, hw, hw), 6)
    y = p.maxpool(p.conv(-1, 16, 3), 3, 2, 1)
    y = p.gap(p.conv(y, 16, 3))
    p.new_unit()
    p.linear(y, 6)
    p.assign_blocks([1, 2])
    for seed in range(60, 90):      # a seed without tied maxima
        x, img, _ = grid_inputs(o, seed, 3)
        if R.kink_margin(o, x, img) > 0:
            return check_step(o, p, 3, seed=seed)
    pytest.fail("every seed has a tie")


def _wide(c, n_classes=10):
    m = PM.Model("wide", (3, 4, 4), n_classes)
    x = m.conv(-1, c, 3)
    m.new_unit()
    x = m.conv(x, 2 * c, 3)
    m.new_unit()
    m.linear(m.gap(m.conv(x, 2 * c, 3)), n_classes)
    return m.assign_blocks([1, 2, 3])


@pytest.mark.parametrize("c", [60, 80, 160, 220, 256], ids=["0.8MB", "1.4MB", "5MB", "10MB", "14MB"])
def test_large_copies_to_the_host(c):
    """Parameters on both sides of 1 MB, from which copies go through pinned
    slots, and of 5, 10 and 14 MB (two, three and four threads, several slots
    a copy): every entry arrives, a block's gradient is the full one's
    and zero elsewhere (the last block's begins inside a thread's part), and
    copies of two contexts from two threads at once (one of them finds the
    pinned slots in use) agree."""
    m = _wide(c)
    assert (m.d * 4 >> 20 > 0) == (c > 60) and (m.d * 4 >> 22) == {160: 1, 220: 2, 256: 3}.get(c, 0)
    rng = np.random.default_rng(3)
    xs = [(rng.standard_normal(m.d) * 0.05).astype(np.float32) for _ in range(2)]
    img, lab = synth.images(4, 2, 3, 4, 4), synth.labels(4, 2, 10)
    with lpp.Context(m, K=1, batch=2) as a, lpp.Context(m, K=1, batch=2) as b:
        for ctx, x in ((a, xs[0]), (b, xs[1])):
            ctx.set_params(x)
            assert np.array_equal(ctx.get_params(0), x)
        i, t = dev(img, lab)
        torch.cuda.synchronize()
        a.step(0, i, t, 0, 0.0)
        full = a.get_grad(0)
        assert np.any(full)
        for part in (1, 2, 3):
            a.step(0, i, t, part, 0.0)
            got, (lo, hi) = a.get_grad(0), a.block_range(part)
            assert hi > lo and np.array_equal(got[lo:hi], full[lo:hi])
            assert not np.any(got[:lo]) and not np.any(got[hi:])
        bad = []

        def read(ctx, x):
            for _ in range(20):
                if not np.array_equal(ctx.get_params(0), x):
                    bad.append(1)

        th = [threading.Thread(target=read, args=c) for c in ((a, xs[0]), (b, xs[1]))]
        for h in th:
            h.start()
        for h in th:
            h.join()
        assert not bad


# bf16 sources whose channels are no multiple of 32: on small grids each thread
# of the load pipeline keeps the tap of its own chunk (the last case's first
# pass has more than 512 workgroups: staged through registers)
@pytest.mark.parametrize("case", [
    (3, 24, 40, 3, 1, 1, 11, 3),
    (3, 40, 136, 3, 2, 1, 13, 2),     # stride-2 data gradient, two column tiles
    (8, 136, 72, 1, 1, 0, 9, 3),
    (3, 48, 16, 7, 2, 3, 17, 2),
    (24, 72, 200, 3, 1, 1, 6, 2),
    (3, 24, 40, 3, 1, 1, 58, 12),
], ids=lambda c: "x".join(map(str, c)))
def test_bf16_channels_in_eights(case):
    from tests.test_gpu_bf16 import test_bf16_conv_passes
    test_bf16_conv_passes(case)


# cin, c1, k, stride, hw, batch: one infinite pixel in an image's last column
@pytest.mark.parametrize("case", [
    (3, 16, 3, 1, 13, 3),
    (3, 32, 7, 2, 25, 2),
    (16, 16, 3, 1, 13, 3),
    (16, 32, 3, 1, 30, 5),
    (20, 16, 3, 1, 58, 12),
    (16, 32, 3, 2, 25, 2),
], ids=lambda c: "x".join(map(str, c)))
def test_weight_gradient_keeps_an_infinity_in_its_place(case):
    """An infinite input pixel that every output clips (its weights are
    negative, a ReLU follows) reaches the weight-gradient entries of its own
    channel and of the taps that read it, and no other entry: those are bit
    for bit what a large finite pixel leaves.  Slots of a box that hold no
    output pixel lie right of the last column and must not read it."""
    cin, c1, k, st, hw, n = case
    pad = k // 2
    o, p = T.twin_conv_net(cin, c1, k, st, pad, 16, hw)
    x, img, lab = grid_inputs(o, 11, n)
    w = x[:c1 * cin * k * k].reshape(c1, cin, k, k)
    w[:, 0] = -np.abs(w[:, 0]) - 0.25
    row, col = hw // 2, hw - 1
    taps = np.zeros((k, k), bool)
    for r in range(k):
        for s in range(k):
            h, v = row + pad - r, col + pad - s
            ho = (hw + 2 * pad - k) // st + 1
            taps[r, s] = h % st == 0 and v % st == 0 and 0 <= h // st < ho and 0 <= v // st < ho
    assert taps.any() and not taps.all()
    grads = []
    for value in (2.0 ** 20, np.inf):
        img[n - 1, 0, row, col] = value
        with lpp.Context(p, K=1, batch=n) as ctx:
            ctx.set_params(x)
            i, t = dev(img, lab)
            torch.cuda.synchronize()
            ctx.step(0, i, t, 0, 0.0)
            assert np.all(np.isfinite(ctx.get_logits(0)))
            grads.append(ctx.get_grad(0))
    reached = np.zeros((c1, cin, k, k), bool)
    reached[:, 0] = taps
    same = np.ones(grads[0].size, bool)
    same[:reached.size] = ~reached.ravel()
    assert np.all(np.isfinite(grads[0]))
    assert np.array_equal(grads[0][same], grads[1][same])


# cin, cout, k, hw, batch: many boxes to a workgroup
@pytest.mark.parametrize("case", [(128, 128, 3, 32, 64), (64, 64, 3, 28, 100), (4, 64, 3, 64, 64), (4, 64, 3, 50, 90),
                                  (64, 64, 1, 32, 60), (64, 64, 1, 28, 80)],
                         ids=lambda c: "x".join(map(str, c)))
def test_weight_gradient_error_does_not_grow_with_the_tensor(case):
    """Against 64-bit sums over the pass's own operands.  n additions of
    random terms in a row round to 2^-24 sqrt(n / 6) of the root of the terms'
    squares; n is 16, where rows are no power of two long 64.  What follows in fp32 (four waves,
    the splits) rounds the sum itself: 2^-24 of it.  A quarter on top."""
    cin, c1, k, hw, n = case
    o, p = T.twin_conv_net(cin, c1, k, 1, k // 2, 16, hw)
    g = torch.Generator("cuda").manual_seed(3)
    img = torch.randn((n, cin, hw, hw), generator=g, device="cuda")
    lab = torch.randint(6, (n,), generator=g, device="cuda", dtype=torch.int32)
    with lpp.Context(p, K=1, batch=n) as ctx:
        ctx.set_params(T.init_x(o.specs, 5).astype(np.float32))
        torch.cuda.synchronize()
        ctx.step(0, img, lab, 0, 0.0)
        got = ctx.get_grad(0)[:c1 * cin * k * k].reshape(c1, cin, k, k)
        dy = torch.from_numpy(ctx.get_activation_grad(0, 0, (c1, hw, hw))).cuda().double()
    d = dy.permute(1, 0, 2, 3).reshape(c1, -1).contiguous()
    pad = torch.nn.functional.pad(img.double(), (k // 2,) * 4)
    ref = np.empty(got.shape)
    sq = np.empty(got.shape)
    for r in range(k):
        for s in range(k):
            v = pad[:, :, r:r + hw, s:s + hw].permute(0, 2, 3, 1).reshape(-1, cin).contiguous()
            ref[:, :, r, s] = (d @ v).cpu().numpy()
            sq[:, :, r, s] = (d.square() @ v.square()).cpu().numpy()
    u, chain = 2.0 ** -24, 16 if hw & (hw - 1) == 0 else 64
    err = np.sqrt(np.mean((got - ref) ** 2 / sq))
    bound = 1.25 * u * np.sqrt(chain / 6 + np.mean(ref ** 2 / sq))
    print(case, "error %.3e, bound %.3e" % (err, bound), file=sys.stderr, flush=True)
    assert err < bound


def _repeated_batch(o, p, small, times, dtype=lpp.FP32):
    """Logits and gradient of a batch without batch norm, and of the same
    images `times` times over, whose activations are larger than a buffer
    descriptor reaches."""
    g = torch.Generator("cuda").manual_seed(3)
    img = torch.randn((small,) + o.in_shape, generator=g, device="cuda")
    lab = torch.randint(o.n_classes, (small,), generator=g, device="cuda", dtype=torch.int32)
    out = []
    for k in (1, times):
        with lpp.Context(p, K=1, batch=small * k, dtype=dtype) as ctx:
            ctx.set_params(T.init_x(o.specs, 5).astype(np.float32))
            i, t = img.repeat(k, 1, 1, 1), lab.repeat(k)
            torch.cuda.synchronize()
            ctx.step(0, i, t, 0, 0.0)
            out.append((ctx.get_logits(0), ctx.get_grad(0)))
        del i, t
        torch.cuda.empty_cache()
    return out


# over 2 GiB: a stem's output and a 3x3 conv's operands; a stride-2 conv's operands
@pytest.mark.parametrize("net,times", [
    (T.twin_conv_net(4, 16, 3, 1, 1, 16, 64), 1125),
    (T.twin_conv2_net(4, 16, 32, 3, 2, 1, 96), 1000),
], ids=["stride1", "stride2"])
def test_tensors_over_2_gib(net, times):
    (logits, grad), (many, mean) = _repeated_batch(*net, 8, times)
    assert np.array_equal(many, np.tile(logits, (times, 1)))
    err = np.linalg.norm(mean.astype(np.float64) - grad) / np.linalg.norm(grad)
    assert err < 1e-5, err


def test_bf16_tensors_over_2_gib():
    """The load pipeline of sources of 32k channels reads through a buffer
    descriptor, which yields zeros past 2 GiB: such a source takes the path
    through registers."""
    (logits, grad), (many, mean) = _repeated_batch(*T.twin_conv_net(8, 64, 3, 1, 1, 64, 64), 8, 520, dtype=lpp.BF16)
    # (one rounding of a stored value may fall the other way: 2^-8 of it, one of 4096 that the pool averages)
    assert np.max(np.abs(many - np.tile(logits, (520, 1)))) < 1e-5 * np.max(np.abs(logits))
    err = np.linalg.norm(mean.astype(np.float64) - grad) / np.linalg.norm(grad)
    assert err < 2e-2, err


@pytest.mark.parametrize("hw", [13, 14])
def test_maxpool_gradient_added_to_another(hw):
    """A map that a max pool 3x3/2 and, later, a stride-2 conv read: the
    pool's gradient is added to the conv's.  Argmax decisions on identical
    values (exact grid)."""
    o = OM.Net("poolnet", 3, hw, hw, 6)
    x = o.conv(-1, 3, 16, 3, 1, 1)
    a = o.maxpool(x, 3, 2, 1)
    a = o.gap(o.add(a, o.conv(x, 16, 16, 3, 2, 1)))
    o.next_unit()
    o.linear(a, 16, 6)
    o.set_blocks([1, 2])
    p = PM.Model("poolnet", (3, hw, hw), 6)
    y = p.conv(-1, 16, 3)
    z = p.maxpool(y, 3, 2, 1)
    z = p.gap(p.add(z, p.conv(y, 16, 3, 2)))
    p.new_unit()
    p.linear(z, 6)
    p.assign_blocks([1, 2])
    for seed in range(60, 90):      # a seed without tied maxima
        x, img, _ = grid_inputs(o, seed, 3)
        if R.kink_margin(o, x, img) > 0:
            return check_step(o, p, 3, seed=seed)
    pytest.fail("every seed has a tie")


@pytest.mark.parametrize("mode", [lpp.SEQUENTIAL, lpp.ASYNC], ids=["sequential", "async"])
def test_bf16_relu_decision_recomputed(mode):
    """The BN backward's sums decide the ReLU from the BN input, rounded to
    bf16 as the stored output: the same decision for every entry, also where
    outputs lie about half of the smallest bf16 number (scales of 1e-40) and
    round to zero, and where they are all zero."""
    n, hw, c = 4, 8, 16
    m = PM.Model("bn", (8, hw, hw), 6)
    y = m.maxpool(m.conv(-1, c, 3), 3, 2, 1)
    r = m.relu(m.bn(y))
    y = m.conv(r, 16, 3)
    m.new_unit()
    m.linear(m.gap(y), 6)
    m.assign_blocks([1, 2])
    x = T.init_x(m.specs, 5).astype(np.float32)
    lo = c * 8 * 9                   # gamma, beta
    x[lo:lo + 2 * c] = 0
    x[lo:lo + c] = np.array([1.0, 1e-40, 0.0, -1e-40] * (c // 4), np.float32)
    x[lo + c] = 0.3
    g = torch.Generator("cuda").manual_seed(3)
    img = torch.randn((n, 8, hw, hw), generator=g, device="cuda")
    lab = torch.randint(6, (n,), generator=g, device="cuda", dtype=torch.int32)
    with lpp.Context(m, K=1, batch=n, mode=mode, dtype=lpp.BF16) as ctx:
        ctx.set_params(x)
        torch.cuda.synchronize()
        ctx.step(0, img, lab, 0, 0.0)
        out = ctx.get_activation(0, r, (c, 4, 4))
        dy = ctx.get_activation_grad(0, r, (c, 4, 4)).astype(np.float64)
        got = ctx.get_grad(0)[lo + c:lo + 2 * c]
    assert np.any(out[:, 1] > 0) and np.any(out[:, 1] == 0) and not np.any(out[:, 2])
    masked = np.where(out > 0, dy, 0.0)
    # a decision that differs moves its channel's sum by a term, 1/64 of their magnitudes and more
    assert np.all(np.abs(got - masked.sum((0, 2, 3))) <= 1e-5 * np.abs(dy).sum((0, 2, 3)))
