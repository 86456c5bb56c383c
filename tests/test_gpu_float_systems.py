"""GPU parity of the paper's two floating-point comparison systems (FloatRS-quant, FloatRS-fp) against
the CPU oracle on the same seeded inputs.  The binary32 noise, the rounded inputs and everything the
int8 network computes from them are bit-exact; the fp32 network is compared with the oracle's
binary64 evaluation of the same network within a tolerance derived from fp32 summation, and its
class decisions wherever the oracle's margin exceeds that tolerance."""
import ctypes

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

QUANT, FP = oracle.FLOATRS_QUANT, oracle.FLOATRS_FP
ALPHA = 0.001
# fp32 network against the binary64 oracle: every tensor element within REL of the tensor's largest
# magnitude.  A convolution sums K <= 4608 products in fp32 (relative error of a sum about sqrt(K) u
# typical, K u worst case, u = 2^-24 = 6e-8) and the nets are up to 110 layers deep with gains near 1:
# sqrt(110) * sqrt(4608) * u = 4e-5 if every layer erred in the same direction at its typical size.
# Measured on the workloads: 3e-7 (ResNet-20) to 1.2e-6 (ResNet-50) of the largest logit.
REL = 1e-4


@pytest.fixture(scope="module")
def isr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_09413_amd as lib
    return lib


def _load(isr, blob, chunk):
    m = isr.isr_load_model(blob)
    isr.isr_set_workspace(m, chunk, float_fp=True)
    return m


def _say(msg):
    print(msg, flush=True)


@pytest.mark.parametrize("sigma", [0.0, 0.4, 31.875, 127.5, 255.0])
def test_continuous_noise_is_bit_exact_cifar_shape(isr, sigma):
    _say(f"float noise parity 32x32 sigma={sigma}")
    m = _load(isr, synth.build_model(0), 64)
    x = synth.make_image(0, 1)
    for seed, image, phase, begin, count in ((0, 0, 0, 0, 5), (0x0123456789ABCDEF, 7, 1, 99990, 9)):
        got_q = isr.isr_float_debug_noisy(m, x, sigma, seed, image, phase, begin, count, QUANT)
        got_f = isr.isr_float_debug_noisy(m, x, sigma, seed, image, phase, begin, count, FP)
        assert got_q.dtype == np.int8 and got_f.dtype == np.float32
        for s in range(count):
            want_f = oracle.noisy_float(x, sigma, seed, image, phase, begin + s)
            assert np.array_equal(got_f[s].view(np.uint32), want_f.view(np.uint32)), (sigma, seed, s)
            assert np.array_equal(got_q[s], oracle.noisy_quant(x, sigma, seed, image, phase, begin + s)), (sigma, seed, s)
    m.close()


def test_continuous_noise_is_bit_exact_224_shape_and_extreme_pixels(isr):
    _say("float noise parity 224x224")
    m = _load(isr, synth.build_model(3), 8)
    x = synth.make_image(3, 1)
    x[0, :8, :] = 0
    x[1, :8, :] = 255
    for sigma in (63.75, 255.0):
        got_q = isr.isr_float_debug_noisy(m, x, sigma, 5, 3, 1, 12345, 2, QUANT)
        got_f = isr.isr_float_debug_noisy(m, x, sigma, 5, 3, 1, 12345, 2, FP)
        for s in range(2):
            assert np.array_equal(got_f[s].view(np.uint32), oracle.noisy_float(x, sigma, 5, 3, 1, 12345 + s).view(np.uint32))
            assert np.array_equal(got_q[s], oracle.noisy_quant(x, sigma, 5, 3, 1, 12345 + s))
    m.close()


@pytest.mark.parametrize("cfg,size,chunk,count", [(0, None, 24, 70), (1, None, 64, 150), (3, 64, 16, 20)])
def test_floatrs_quant_logits_and_votes_are_bit_exact(isr, cfg, size, chunk, count):
    """Several chunks and a ragged last one; sample range not starting at 0."""
    _say(f"FloatRS-quant parity config {cfg}")
    blob = synth.build_model(cfg) if size is None else synth.build_model(cfg, size=size)
    m = _load(isr, blob, chunk)
    om = oracle.Model(blob)
    x = synth.make_image(cfg, 2) if size is None else synth.make_image(cfg, 2, shape=(3, size, size))
    for sigma, seed, image, phase, begin in ((63.75, 11, 2, 0, 0), (127.5, 0xABCDEF0123, 5, 1, 1000)):
        lg, am, cnt = isr.isr_float_debug_forward(m, x, sigma, seed, image, phase, begin, count, QUANT)
        wl, wa, wc = om.mc_float(x, sigma, seed, image, phase, begin, count, QUANT)
        assert np.array_equal(lg, wl) and np.array_equal(am, wa) and np.array_equal(cnt, wc)
    m.close()


def _check_fp_logits(got, want, got_argmax):
    """Logits within REL of the sample's largest magnitude; the class equals the oracle's wherever the
    oracle's top-two margin exceeds twice that tolerance, and is a near-tie of the oracle's otherwise."""
    ambiguous = 0
    for s in range(want.shape[0]):
        tol = REL * np.abs(want[s]).max()
        assert np.all(np.abs(got[s].astype(np.float64) - want[s]) <= tol), (s, np.abs(got[s] - want[s]).max(), tol)
        order = np.argsort(-want[s], kind="stable")
        margin = want[s][order[0]] - want[s][order[1]]
        if margin > 2 * tol:
            assert got_argmax[s] == order[0], s
        else:
            ambiguous += 1
            assert want[s][got_argmax[s]] >= want[s][order[0]] - 2 * tol, s
        assert got_argmax[s] == int(np.argmax(got[s])), s          # the vote kernel against the logits it read
    return ambiguous


@pytest.mark.parametrize("cfg,size,chunk,count", [(0, None, 64, 40), (1, None, 128, 70), (2, None, 32, 20), (3, 64, 32, 20)])
def test_floatrs_fp_logits_within_fp32_tolerance(isr, cfg, size, chunk, count):
    _say(f"FloatRS-fp parity config {cfg}")
    blob = synth.build_model(cfg) if size is None else synth.build_model(cfg, size=size)
    m = _load(isr, blob, chunk)
    assert 1 <= isr.isr_float_chunk(m, FP) <= chunk // 4 and count > 2 * isr.isr_float_chunk(m, FP)
    om = oracle.Model(blob)
    x = synth.make_image(cfg, 3) if size is None else synth.make_image(cfg, 3, shape=(3, size, size))
    worst = 0.0
    for sigma, seed, image, phase, begin in ((63.75, 11, 2, 0, 0), (127.5, 0xABCDEF0123, 5, 1, 1000)):
        lg, am, cnt = isr.isr_float_debug_forward(m, x, sigma, seed, image, phase, begin, count, FP)
        wl, wa, wc = om.mc_float(x, sigma, seed, image, phase, begin, count, FP)
        assert lg.dtype == np.float32
        amb = _check_fp_logits(lg, wl, am)
        assert np.array_equal(cnt, np.bincount(am, minlength=om.classes))
        assert np.abs(cnt.astype(np.int64) - wc.astype(np.int64)).sum() <= 2 * amb
        worst = max(worst, float((np.abs(lg - wl).max(axis=1) / np.abs(wl).max(axis=1)).max()))
    _say(f"  largest logit deviation / largest logit: {worst:.2e}")
    m.close()


@pytest.mark.parametrize("cfg,size", [(0, None), (1, None), (3, 64)])
def test_floatrs_fp_layer_tensors(isr, cfg, size):
    """Every tensor the fp32 kernels store, one noisy copy, against the oracle's float network."""
    _say(f"FloatRS-fp layer tensors config {cfg}")
    blob = synth.build_model(cfg) if size is None else synth.build_model(cfg, size=size)
    m = _load(isr, blob, 16)
    om = oracle.Model(blob)
    x = synth.make_image(cfg, 4) if size is None else synth.make_image(cfg, 4, shape=(3, size, size))
    sigma, seed, image, phase, sample = 63.75, 21, 1, 1, 77
    _, want = om.forward_float(oracle.noisy_float(x, sigma, seed, image, phase, sample))
    checked = skipped = 0
    for tid in range(om.n_tensors - 1):
        c, h, w, _ = om.tensor_shape(tid)
        try:
            got = isr.isr_float_debug_tensor(m, x, sigma, seed, image, phase, sample, tid, (c, h, w))
        except isr.IsrError as e:
            assert e.status == isr.ISR_ERR_UNSUPPORTED      # convolution output folded into the add after it
            skipped += 1
            continue
        tol = REL * max(np.abs(want[tid]).max(), 1e-30)
        assert np.all(np.abs(got.astype(np.float64) - want[tid]) <= tol), (tid, np.abs(got - want[tid]).max(), tol)
        checked += 1
    assert checked >= 3 and checked > skipped
    m.close()


@pytest.mark.parametrize("copies", [1, 9, 40, 80])
def test_floatrs_fp_every_tile_and_addressing_form(isr, copies):
    """The fp32 convolution on every tile its launcher picks (few to many pixels), with plain, tap-wise and table
    addressing, on maps whose pixels and channels divide no tile; the last copies' logits against the oracle."""
    _say(f"FloatRS-fp tiles, {copies} copies")
    from synth.models import NetBuilder
    b = NetBuilder(rng=np.random.default_rng(81), in_shape=(3, 43, 44), num_classes=6)
    t0 = b.tensor(3, 43, 44, 0, 74.0)
    t = b.conv(t0, 128, 3, 1, 1, True)           # table: 4 stored channels, 128-channel tiles
    u = b.conv(t, 128, 3, 1, 1, True)            # tap by tap
    u = b.conv(u, 128, 1, 1, 0, False)           # plain, fused add
    t = b.add(t, u, True)
    t = b.conv(t, 64, 1, 1, 0, True)
    t = b.conv(t, 48, 5, 2, 2, True)             # 64-channel tiles, 48 of them real; stride 2
    t = b.conv(t, 80, 3, 1, 0, True)             # table: a step of 32 spans taps; unpadded
    t = b.conv(t, 32, 1, 2, 0, True)
    t = b.conv(t, 16, 3, 1, 1, True)
    b.fc(b.gap(t), 6)
    blob = b.blob()
    m = _load(isr, blob, 4 * copies)
    om = oracle.Model(blob)
    x = np.random.default_rng(5).integers(0, 256, size=(3, 43, 44)).astype(np.uint8)
    lg, am, cnt = isr.isr_float_debug_forward(m, x, 63.75, 3, 1, 1, 50, copies, FP)
    k = min(copies, 3)
    wl = om.mc_float(x, 63.75, 3, 1, 1, 50 + copies - k, k, FP)[0]
    _check_fp_logits(lg[-k:], wl, am[-k:])
    assert cnt.sum() == copies
    m.close()


@pytest.mark.parametrize("copies", [1, 60])
@pytest.mark.parametrize("closing_first", [False, True])
def test_floatrs_fp_residual_computed_in_the_kernel(isr, closing_first, copies):
    """First blocks of a stage, whose residual is a projection that only their add reads: closing convolution and projection in
    one kernel, in either order, with 1 to 5 steps each (fewer and more than stages), strides 1 and 2, channels that fill no tile,
    ReLU on the inner convolution; the results that are no longer stored remain to be had one by one."""
    _say(f"FloatRS-fp paired 1x1 layers, {copies} copies")
    from synth.models import NetBuilder
    b = NetBuilder(rng=np.random.default_rng(84), in_shape=(3, 29, 28), num_classes=6)
    t = b.conv(b.tensor(3, 29, 28, 0, 74.0), 32, 3, 1, 1, True)
    inner = []
    for mid, out, stride, relu in ((32, 128, 1, False), (160, 144, 2, True), (64, 400, 1, False)):
        u = b.conv(t, mid, 3, stride, 1, True)
        if closing_first:
            u = b.conv(u, out, 1, 1, 0, relu)
            inner.append(u)
            t = b.add(u, b.conv(t, out, 1, stride, 0, False), True)
        else:
            r = b.conv(t, out, 1, stride, 0, relu)
            inner.append(r)
            t = b.add(b.conv(u, out, 1, 1, 0, False), r, True)
        t = b.conv(t, 96, 1, 1, 0, True)
    b.fc(b.gap(t), 6)
    blob = b.blob()
    m = _load(isr, blob, 4 * copies)
    om = oracle.Model(blob)
    x = np.random.default_rng(5).integers(0, 256, size=(3, 29, 28)).astype(np.uint8)
    lg, am, cnt = isr.isr_float_debug_forward(m, x, 63.75, 3, 1, 1, 50, copies, FP)
    k = min(copies, 3)
    wl = om.mc_float(x, 63.75, 3, 1, 1, 50 + copies - k, k, FP)[0]
    _check_fp_logits(lg[-k:], wl, am[-k:])
    assert cnt.sum() == copies
    _, want = om.forward_float(oracle.noisy_float(x, 63.75, 3, 1, 1, 50))
    for tid in inner:
        c, h, w, _ = om.tensor_shape(tid)
        got = isr.isr_float_debug_tensor(m, x, 63.75, 3, 1, 1, 50, tid, (c, h, w))
        assert np.all(np.abs(got.astype(np.float64) - want[tid]) <= REL * np.abs(want[tid]).max()), tid
    m.close()


def test_floatrs_fp_pairs_of_few_tiles_run_apart(isr):
    """A closing layer and its projection as two kernels up to 127 tiles of 128 x 128, as one beyond, which writes the same bits."""
    _say("FloatRS-fp pairs of few tiles")
    from synth.models import NetBuilder
    b = NetBuilder(rng=np.random.default_rng(86), in_shape=(3, 30, 28), num_classes=6)
    t = b.conv(b.tensor(3, 30, 28, 0, 74.0), 64, 3, 1, 1, True)
    u = b.conv(t, 96, 3, 2, 1, True)
    r = b.conv(t, 496, 1, 2, 0, True)
    t = b.add(b.conv(u, 496, 1, 1, 0, False), r, True)   # 15 x 14 pixels, four tiles of channels
    b.fc(b.gap(t), 6)
    m = _load(isr, b.blob(), 4 * 20)
    x = np.random.default_rng(6).integers(0, 256, size=(3, 30, 28)).astype(np.uint8)
    logits = {}
    for copies, together in ((1, False), (18, False), (19, True)):   # 8, 120, 128 tiles
        isr.isr_profile(m, 1)
        logits[copies] = isr.isr_float_debug_forward(m, x, 63.75, 3, 1, 1, 50, copies, FP)[0]
        assert any("pair" in k["name"] for k in isr.isr_profile_read(m)) == together
    assert np.array_equal(logits[1], logits[19][:1]) and np.array_equal(logits[18], logits[19][:18])
    m.close()


def test_floatrs_fp_joined_layers_each_where_the_workspace_has_room(isr):
    """A first layer with its pooling, and sums one of whose readers has no room beside it (256 channels next to 128): in a workspace
    of the size asked for the first layer and its pooling are joined alone, in twice that all; the logits are the same to the bit."""
    _say("FloatRS-fp joined layers and the workspace")
    import torch
    from synth.models import NetBuilder
    b = NetBuilder(rng=np.random.default_rng(87), in_shape=(3, 32, 28), num_classes=6)
    t = b.maxpool(b.conv(b.tensor(3, 32, 28, 0, 74.0), 64, 7, 2, 3, True), 3, 2, 1)   # 8 x 7 pixels
    r = b.conv(t, 128, 1, 1, 0, True)
    t = b.add(b.conv(b.conv(r, 64, 1, 1, 0, True), 128, 1, 1, 0, False), r, True)
    t = b.add(b.conv(b.conv(t, 128, 1, 1, 0, True), 128, 1, 1, 0, False), t, True)
    t = b.conv(t, 256, 1, 1, 0, True)
    b.fc(b.gap(t), 6)
    chunk, copies = 4 * 900, 900
    m = _load(isr, b.blob(), chunk)
    bytes_ = isr.lib().isr_float_workspace_bytes(m.handle, chunk, FP)
    x = torch.from_numpy(np.random.default_rng(7).integers(0, 256, size=(3, 32, 28)).astype(np.uint8)).cuda()
    room = torch.empty(2 * bytes_ + 256, dtype=torch.uint8, device="cuda")
    logits = []
    for size, kernels in ((bytes_, {"fstem_pool_kernel"}), (2 * bytes_, {"fstem_pool_kernel", "fexpand_kernel<128>", "fexpand_kernel<256>"})):
        at = (room.data_ptr() + 255) // 256 * 256
        isr._check(isr.lib().isr_set_workspace(m.handle, ctypes.c_void_p(at), size, chunk, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)), "isr_set_workspace")
        isr.isr_profile(m, 1)
        logits.append(isr.isr_float_debug_forward(m, x, 63.75, 3, 1, 1, 50, copies, FP)[0])
        names = {k["name"] for k in isr.isr_profile_read(m)}
        assert {n for n in names if n.startswith(("fstem_pool", "fexpand"))} == kernels, names
    assert np.array_equal(logits[0], logits[1])
    m.close()


@pytest.mark.parametrize("copies", [150, 305])
@pytest.mark.parametrize("mid,out,reduced,pair", [(64, 128, 64, 0), (96, 512, 64, 0), (64, 384, 128, 0), (256, 512, 128, 0), (64, 128, 256, 0), (64, 384, 256, 0), (160, 1024, 256, 0),
                                                  (32, 128, 64, 1), (96, 512, 64, 2), (64, 512, 128, 1), (160, 256, 128, 2)])
def test_floatrs_fp_closing_layer_and_the_reader_of_its_sum(isr, mid, out, reduced, pair, copies):
    """A block's closing 1x1 layer with its add and the 1x1 layer that reads the sum: one kernel for many copies (nearly a round of
    workgroups and nearly two, whose pixels fill no tile; one and more steps of the first layer, one to eight times 128 channels), two for one copy.  pair: the residual is a
    projection of that stride, computed in the kernel as well.  Where 256 channels of result next to a sum of 128 are more than the
    workspace was ever asked for, two kernels.  The logits are the same to the bit and near the oracle's."""
    _say(f"FloatRS-fp closing layer {mid} -> {out} -> {reduced}, projection {pair}, {copies} copies")
    from synth.models import NetBuilder
    b = NetBuilder(rng=np.random.default_rng(85), in_shape=(3, 29, 28), num_classes=6)
    t = b.conv(b.tensor(3, 29, 28, 0, 74.0), 32, 3, 1 if pair == 2 else 2, 1, True)
    if pair:
        u = b.conv(t, mid, 3, pair, 1, True)
        r = b.conv(t, out, 1, pair, 0, True)   # issued right before the closing layer, which takes it along
        t = b.add(b.conv(u, out, 1, 1, 0, False), r, True)
    else:
        t = b.conv(t, out, 1, 1, 0, True)
        t = b.add(b.conv(b.conv(t, mid, 1, 1, 0, True), out, 1, 1, 0, False), t, True)
    u = b.conv(t, reduced, 1, 1, 0, True)                      # reads the sum, as the next add does
    t = b.add(b.conv(u, out, 1, 1, 0, True), t, False)
    t = b.conv(t, reduced, 1, 1, 0, False)
    b.fc(b.gap(t), 6)
    blob = b.blob()
    m = _load(isr, blob, 4 * copies)
    om = oracle.Model(blob)
    x = np.random.default_rng(5).integers(0, 256, size=(3, 29, 28)).astype(np.uint8)
    isr.isr_profile(m, 1)
    lg, am, cnt = isr.isr_float_debug_forward(m, x, 63.75, 3, 1, 1, 50, copies, FP)
    names = [k["name"] for k in isr.isr_profile_read(m) if k["name"].startswith("fexpand_kernel")]
    assert bool(names) == (reduced <= out and (reduced < 256 or copies > 300))
    assert any("pair" in n for n in names) == bool(pair)
    for i in (0, 1, copies // 2, copies - 1):
        assert np.array_equal(isr.isr_float_debug_forward(m, x, 63.75, 3, 1, 1, 50 + i, 1, FP)[0][0], lg[i]), i
    k = 2
    wl = om.mc_float(x, 63.75, 3, 1, 1, 50 + copies - k, k, FP)[0]
    _check_fp_logits(lg[-k:], wl, am[-k:])
    assert cnt.sum() == copies
    m.close()


@pytest.mark.parametrize("h,w,copies", [(9, 63, 5), (9, 64, 5), (3, 32, 9), (40, 31, 2), (17, 16, 9), (15, 15, 300), (16, 15, 3), (1, 15, 40), (5, 1, 40), (1, 1, 3)])
def test_floatrs_fp_3x3_layers_from_one_run_of_pixels(isr, h, w, copies):
    """3x3 layers whose nine taps are read from one run of pixels in LDS: the widest maps of each size of run (15, 31, 63) and the next
    (64: tap by tap), single rows, columns and pixels, tiles that span images, 32 to 160 channels in and out, few tiles and many,
    with a residual and without, against the oracle."""
    _say(f"FloatRS-fp 3x3 layers on {h} x {w}, {copies} copies")
    from synth.models import NetBuilder
    k = 4 - (w - 1) % 4                                         # inputs are a multiple of 4 pixels wide
    b = NetBuilder(rng=np.random.default_rng(86), in_shape=(3, h + k - 1, w + k - 1), num_classes=6)
    t = b.conv(b.tensor(3, h + k - 1, w + k - 1, 0, 74.0), 32, k, 1, 0, True)
    t = b.conv(t, 96, 3, 1, 1, True)
    u = b.conv(t, 64, 3, 1, 1, True)
    t = b.add(b.conv(u, 96, 3, 1, 1, False), t, True)
    t = b.conv(t, 160, 3, 1, 1, True)
    t = b.conv(t, 32, 3, 1, 1, False)
    b.fc(b.gap(t), 6)
    blob = b.blob()
    m = _load(isr, blob, 4 * copies)
    om = oracle.Model(blob)
    x = np.random.default_rng(5).integers(0, 256, size=(3, h + k - 1, w + k - 1)).astype(np.uint8)
    lg, am, cnt = isr.isr_float_debug_forward(m, x, 63.75, 3, 1, 1, 50, copies, FP)
    n = min(copies, 3)
    wl = om.mc_float(x, 63.75, 3, 1, 1, 50 + copies - n, n, FP)[0]
    _check_fp_logits(lg[-n:], wl, am[-n:])
    assert np.array_equal(isr.isr_float_debug_forward(m, x, 63.75, 3, 1, 1, 50 + copies // 2, 1, FP)[0][0], lg[copies // 2])
    assert cnt.sum() == copies
    m.close()


@pytest.mark.parametrize("h,w,copies", [(32, 32, 40), (9, 47, 5), (9, 48, 5), (15, 15, 3), (17, 16, 3), (1, 15, 40), (5, 1, 40), (1, 1, 3)])
def test_floatrs_fp_3x3_layers_of_16_channels_from_one_run_of_pixels(isr, h, w, copies):
    """The same for inputs of 16, 48 and 80 channels, whose taps need no barrier between them: widest maps of both sizes of run (15, 47)
    and the next (16, 48: from the table), into 16 to 144 channels, with a residual and without."""
    _say(f"FloatRS-fp 3x3 layers of 16 channels on {h} x {w}, {copies} copies")
    from synth.models import NetBuilder
    k = 4 - (w - 1) % 4
    b = NetBuilder(rng=np.random.default_rng(88), in_shape=(3, h + k - 1, w + k - 1), num_classes=6)
    t = b.conv(b.tensor(3, h + k - 1, w + k - 1, 0, 74.0), 16, k, 1, 0, True)
    t = b.add(b.conv(b.conv(t, 16, 3, 1, 1, True), 16, 3, 1, 1, False), t, True)
    t = b.conv(t, 48, 3, 1, 1, True)
    t = b.conv(t, 80, 3, 1, 1, True)
    t = b.conv(t, 144, 3, 1, 1, False)
    b.fc(b.gap(t), 6)
    blob = b.blob()
    m = _load(isr, blob, 4 * copies)
    om = oracle.Model(blob)
    x = np.random.default_rng(5).integers(0, 256, size=(3, h + k - 1, w + k - 1)).astype(np.uint8)
    isr.isr_profile(m, 1)
    lg, am, cnt = isr.isr_float_debug_forward(m, x, 63.75, 3, 1, 1, 50, copies, FP)
    assert any(q["name"].startswith("fpatch16_kernel") for q in isr.isr_profile_read(m)) == (w <= 47)
    n = min(copies, 3)
    wl = om.mc_float(x, 63.75, 3, 1, 1, 50 + copies - n, n, FP)[0]
    _check_fp_logits(lg[-n:], wl, am[-n:])
    assert np.array_equal(isr.isr_float_debug_forward(m, x, 63.75, 3, 1, 1, 50 + copies // 2, 1, FP)[0][0], lg[copies // 2])
    assert cnt.sum() == copies
    m.close()


@pytest.mark.parametrize("h,w,copies", [(224, 224, 2), (64, 64, 5), (37, 28, 3), (30, 44, 3), (9, 8, 4), (150, 124, 2), (17, 128, 2), (3, 4, 2), (33, 252, 2)])
def test_floatrs_fp_first_layer_with_its_pooling(isr, h, w, copies):
    """7x7 / 2 layer into 64 channels and 3x3 / 2 pooling in one kernel: bands and strips that end inside the image and beside it, odd
    sizes, images smaller than a window; the pooled tensor and the layer's own (which the kernel does not store) against the oracle."""
    _say(f"FloatRS-fp first layer with pooling {h} x {w}, {copies} copies")
    from synth.models import NetBuilder
    b = NetBuilder(rng=np.random.default_rng(87), in_shape=(3, h, w), num_classes=6)
    c = b.conv(b.tensor(3, h, w, 0, 74.0), 64, 7, 2, 3, w != 44)
    t = b.maxpool(c, 3, 2, 1)
    u = b.conv(t, 64, 1, 1, 0, True)
    b.fc(b.gap(u), 6)
    blob = b.blob()
    m = _load(isr, blob, 4 * copies)
    om = oracle.Model(blob)
    x = np.random.default_rng(5).integers(0, 256, size=(3, h, w)).astype(np.uint8)
    isr.isr_profile(m, 1)
    lg, am, cnt = isr.isr_float_debug_forward(m, x, 63.75, 3, 1, 1, 50, copies, FP)
    assert any(k["name"] == "fstem_pool_kernel" for k in isr.isr_profile_read(m))
    wl = om.mc_float(x, 63.75, 3, 1, 1, 50, copies, FP)[0]
    _check_fp_logits(lg, wl, am)
    _, want = om.forward_float(oracle.noisy_float(x, 63.75, 3, 1, 1, 50))
    got = [isr.isr_float_debug_tensor(m, x, 63.75, 3, 1, 1, 50, tid, om.tensor_shape(tid)[:3]) for tid in (c, t)]
    for tid, g in zip((c, t), got):
        assert np.all(np.abs(g.astype(np.float64) - want[tid]) <= REL * np.abs(want[tid]).max()), tid
    rows, cols = got[1].shape[1:]
    padded = np.full((64, 2 * rows + 1, 2 * cols + 1), -np.inf, np.float32)
    padded[:, 1:got[0].shape[1] + 1, 1:got[0].shape[2] + 1] = got[0]
    pooled = np.max([padded[:, i:i + 2 * rows:2, j:j + 2 * cols:2] for i in range(3) for j in range(3)], axis=0)
    # the layer's own kernel adds the same products in another order: a few roundings of the largest sum
    assert np.abs(pooled - got[1]).max() <= 2.0 ** -20 * np.abs(pooled).max()
    m.close()


# 2-norm error of the logits that one rounding per product gives (the fp32 matrix instruction, a chain of fused
# multiply-adds), measured over 768 copies: 2.0e-7 and 3.1e-7.  The kernels round less often (1.45e-7 and 2.1e-7); the bounds
# are the chain's error plus 15 % for the spread of 24 copies.  Sums that all err to the same side, as the matrix unit's do
# by themselves, add up over the blocks of the deep net: 5.3e-7.
@pytest.mark.parametrize("cfg,bound", [(1, 2.3e-7), (2, 3.6e-7)])
def test_floatrs_fp_error_is_no_larger_than_that_of_fp32_products(isr, cfg, bound):
    _say(f"FloatRS-fp error against binary64, config {cfg}")
    blob = synth.build_model(cfg)
    m = _load(isr, blob, 128)
    om = oracle.Model(blob)
    x = synth.make_image(cfg, 1)
    lg, _, _ = isr.isr_float_debug_forward(m, x, 64.0, 1, 1, 1, 0, 24, FP)
    wl, _, _ = om.mc_float(x, 64.0, 1, 1, 1, 0, 24, FP)
    rel = np.linalg.norm(lg - wl, axis=1) / np.linalg.norm(wl, axis=1)
    error = float(np.sqrt(np.mean(rel ** 2)))
    _say(f"  relative error of the logits: {error:.2e}")
    assert error <= bound
    m.close()


def test_floatrs_fp_resnet50_full_size(isr):
    """224 x 224 inputs in the benchmarked chunk: a few scattered sample indices of a long run."""
    _say("FloatRS-fp ResNet-50 full size")
    blob = synth.build_model(3)
    m = _load(isr, blob, 668)
    om = oracle.Model(blob)
    x = synth.make_image(3, 1)
    sigma, seed, image, phase = 63.75, 9, 4, 1
    n = 2 * isr.isr_float_chunk(m, FP) + 37
    lg, am, cnt = isr.isr_float_debug_forward(m, x, sigma, seed, image, phase, 0, n, FP)
    idx = [0, 1, isr.isr_float_chunk(m, FP) - 1, isr.isr_float_chunk(m, FP), n - 2, n - 1]
    from concurrent.futures import ThreadPoolExecutor
    with ThreadPoolExecutor(max_workers=len(idx)) as ex:       # one host thread per index (the C oracle releases the GIL)
        wls = list(ex.map(lambda i: om.mc_float(x, sigma, seed, image, phase, i, 1, FP, threads=1)[0], idx))
    for i, wl in zip(idx, wls):
        _check_fp_logits(lg[i:i + 1], wl, am[i:i + 1])
    assert cnt.sum() == n
    m.close()


@pytest.mark.parametrize("system", [QUANT, FP])
def test_float_certify_against_the_oracle(isr, system):
    _say(f"float certify system {system}")
    blob = synth.build_model(1)
    m = _load(isr, blob, 256)
    om = oracle.Model(blob)
    x = synth.make_image(1, 5)
    sigma, n0, n, seed, image = 63.75, 40, 300, 3, 2
    res, c0, c1 = isr.isr_float_certify(m, x, sigma, n0, n, ALPHA, system, seed, image)
    cls, rad, p_l, k, w0, w1 = oracle.certify_float(om, x, sigma, n0, n, ALPHA, system, seed, image)
    assert c0.sum() == n0 and c1.sum() == n and res.radius_int == 0 and res.radius_sq_int == 0
    if system == QUANT:
        assert np.array_equal(c0, w0) and np.array_equal(c1, w1)
    else:
        # a class decision may differ only for samples whose two best logits are within the fp32 tolerance
        for phase, cnt, total, got in ((0, w0, n0, c0), (1, w1, n, c1)):
            wl, _, _ = om.mc_float(x, sigma, seed, image, phase, 0, total, FP)
            top2 = -np.sort(-wl, axis=1)[:, :2]
            amb = int(np.count_nonzero(top2[:, 0] - top2[:, 1] <= 2 * REL * np.abs(wl).max(axis=1)))
            assert np.abs(got.astype(np.int64) - cnt.astype(np.int64)).sum() <= 2 * amb
    # the decision is the host's function of the tallies the device produced (Alg. 1)
    want = oracle.stats.certify_decision(c0, c1, sigma, n, ALPHA)
    assert res.cls == want[0] and res.n_top == want[3]
    assert res.p_lower == pytest.approx(want[2], rel=1e-9) and res.radius == pytest.approx(want[1], rel=1e-9, abs=1e-12)
    if system == QUANT or np.array_equal(c0, w0) and np.array_equal(c1, w1):
        assert res.cls == cls and res.radius == pytest.approx(rad, rel=1e-9, abs=1e-12)
    m.close()


def test_float_entry_points_reject_bad_arguments(isr):
    import torch
    blob = synth.build_model(0)
    m = isr.isr_load_model(blob)
    x = torch.from_numpy(synth.make_image(0, 1)).cuda()
    L = isr.lib()
    res = isr.Result()
    args = lambda sigma, system: (m.handle, ctypes.c_void_p(x.data_ptr()), ctypes.c_float(sigma), 4, 8, 0.01,
                                  ctypes.c_uint64(0), 0, system, ctypes.byref(res), None, None)
    assert L.isr_float_certify(*args(10.0, QUANT)) == isr.ISR_ERR_WORKSPACE       # no workspace yet
    isr.isr_set_workspace(m, 2)                                                    # too small for one fp32 copy
    assert L.isr_float_certify(*args(10.0, FP)) == isr.ISR_ERR_WORKSPACE
    assert L.isr_float_certify(*args(10.0, QUANT)) == isr.ISR_OK
    isr.isr_set_workspace(m, 16, float_fp=True)
    assert L.isr_float_certify(*args(10.0, FP)) == isr.ISR_OK
    for sigma, system in ((-1.0, QUANT), (float("nan"), FP), (5000.0, FP), (10.0, 0), (10.0, 3)):
        assert L.isr_float_certify(*args(sigma, system)) == isr.ISR_ERR_ARG
    assert L.isr_float_chunk(m.handle, FP) == 4 and L.isr_float_chunk(m.handle, QUANT) == 16 and L.isr_float_chunk(m.handle, 7) == 0
    m.close()
