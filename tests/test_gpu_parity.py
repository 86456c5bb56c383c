"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle
on the same seeded inputs.  Integer results (noisy copies, layer tensors,
logits, argmax, votes) must be bit-exact; radii agree to 1e-9 relative."""
import sys

import numpy as np
import pytest

import oracle
import synth
from synth.models import NetBuilder

pytestmark = pytest.mark.gpu

ALPHA = 0.001


@pytest.fixture(scope="module")
def isr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_09413_amd as lib
    return lib


def _load(isr, blob, chunk):
    m = isr.isr_load_model(blob)
    isr.isr_set_workspace(m, chunk)
    return m


def _say(msg):
    print(msg, flush=True)


def _oracle_at(om, x, sigma, seed, image, phase, indices):
    """Oracle logits and argmax of scattered sample indices, one host thread per index."""
    from concurrent.futures import ThreadPoolExecutor
    import os

    def one(i):
        lg, am, _ = om.mc(x, sigma, seed, image, phase, int(i), 1, threads=1)
        return lg[0], int(am[0])
    with ThreadPoolExecutor(max_workers=min(os.cpu_count() or 1, 16)) as ex:
        out = list(ex.map(one, indices))
    return np.stack([o[0] for o in out]), np.array([o[1] for o in out])


# ---- S2: noise -------------------------------------------------------------

@pytest.mark.parametrize("sigma", [1, 32, 64, 128, 256, 1024])
def test_noisy_copies_cifar_shape(isr, sigma):
    _say(f"noise parity 32x32 sigma={sigma}")
    m = _load(isr, synth.build_model(0), 64)
    x = synth.make_image(0, 1)
    for seed, image, phase, begin, count in ((0, 0, 0, 0, 5), (0x0123456789ABCDEF, 7, 1, 99990, 10)):
        got = isr.isr_debug_noisy(m, x, sigma, seed, image, phase, begin, count)
        for s in range(count):
            want = oracle.noisy(x, sigma, seed, image, phase, begin + s)
            assert np.array_equal(got[s], want), (sigma, seed, s)
    m.close()


def test_noisy_copies_224_shape_and_extreme_pixels(isr):
    _say("noise parity 224x224")
    m = _load(isr, synth.build_model(3), 4)
    x = synth.make_image(3, 1)
    x[0, :8, :] = 0
    x[1, :8, :] = 255
    for sigma in (64, 256):
        got = isr.isr_debug_noisy(m, x, sigma, 5, 3, 1, 12345, 2)
        for s in range(2):
            assert np.array_equal(got[s], oracle.noisy(x, sigma, 5, 3, 1, 12345 + s))
    m.close()


@pytest.mark.parametrize("sigma", [1, 32, 256, 1024])
def test_stored_training_noise_bank(isr, sigma):
    """Unsaturated int16 draws for noise sampled ahead of training: bit-exact against
    the oracle for a range of tensors that does not start at 0, a tensor size that
    leaves the last workgroup ragged, and a tiny tensor."""
    _say(f"noise bank parity sigma={sigma}")
    for seed, bank, first, count, d in ((3, 2, 4094, 5, 3 * 32 * 32), (0xFFFFFFFF00000001, 9, 0, 3, 12)):
        got = isr.isr_noise_bank(sigma, seed, bank, first, count, d).cpu().numpy()
        want = oracle.noise_bank(sigma, seed, bank, first, count, d)
        assert got.dtype == np.int16 and np.array_equal(got, want), (sigma, seed)
    import ctypes
    import torch
    buf = torch.empty(64, dtype=torch.int16, device="cuda")
    for bad_sigma, bad_d in ((0, 8), (1025, 8), (sigma, 6), (sigma, 0)):
        rc = isr.lib().isr_noise_bank(bad_sigma, ctypes.c_uint64(0), 0, 0, 1, bad_d, ctypes.c_void_p(buf.data_ptr()), None)
        assert rc == isr.ISR_ERR_ARG
    assert isr.lib().isr_noise_bank(sigma, ctypes.c_uint64(0), 0, 0, 1, 8, None, None) == isr.ISR_ERR_ARG


@pytest.mark.parametrize("sigma", [44, 88, 175, 343, 800])
def test_sampler_guide_tables_of_every_resolution(isr, sigma):
    """One sigma for each number of buckets per octave of the guide tables, enough draws that some meet a threshold's
    leading bits and (large sigma) some lie below all buckets: stored draws and noisy pixels, bit-exact."""
    _say(f"sampler tables sigma={sigma}")
    got = isr.isr_noise_bank(sigma, 77, 3, 5, 70, 3 * 32 * 32).cpu().numpy()
    assert np.array_equal(got, oracle.noise_bank(sigma, 77, 3, 5, 70, 3 * 32 * 32))
    m = _load(isr, synth.build_model(0), 32)
    x = synth.make_image(0, 1)
    got = isr.isr_debug_noisy(m, x, sigma, 78, 9, 0, 3, 32)
    for s in range(32):
        assert np.array_equal(got[s], oracle.noisy(x, sigma, 78, 9, 0, 3 + s))
    m.close()


@pytest.mark.parametrize("d,count", [(252, 300), (256, 1), (256, 9000), (260, 300), (512, 4100), (768, 2800), (3072, 700)])
def test_noise_bank_tensors_of_whole_and_of_ragged_waves(isr, d, count):
    """Tensors of a multiple of 256 draws (a wave's draws lie in one tensor) and others; more waves than one launch holds at
    once, so that each goes on to further tensors: every draw, for a guide table of each workgroup size."""
    _say(f"noise bank d={d} count={count}")
    for sigma in (32, 200, 1000):
        got = isr.isr_noise_bank(sigma, 5, 11, 1000, count, d).cpu().numpy()
        assert np.array_equal(got, oracle.noise_bank(sigma, 5, 11, 1000, count, d)), sigma


@pytest.mark.parametrize("sigma,groups", [(3, 1), (86, 524288), (86, 524289), (169, 524288), (170, 131072), (170, 131073), (1024, 131072)])
def test_small_banks_read_their_guide_from_memory(isr, sigma, groups):
    """Banks of one step a thread and one group of four draws more, tensors of whole waves and ragged ones: the guide is read from
    memory up to there, from LDS beyond."""
    _say(f"small noise bank sigma={sigma} groups={groups}")
    for d in (4, 256 if groups % 64 == 0 else 4 * groups):
        count = 4 * groups // d
        got = isr.isr_noise_bank(sigma, 9, 2, 17, count, d).cpu().numpy()
        assert np.array_equal(got, oracle.noise_bank(sigma, 9, 2, 17, count, d)), d


@pytest.mark.parametrize("sigma", [2, 32])
def test_device_sampler_law_at_scale(isr, sigma):
    """1.5e8 draws of the device sampler (a full stored-noise bank) against Def. 3.3 itself:
    mean, variance and a chi-square over 50 cells with the exact cell probabilities
    (50-digit arithmetic) -- a property of the law, not of the oracle's code."""
    import mpmath as mp
    import torch
    _say(f"sampler law at scale sigma={sigma}")
    count, d = 50000, 3072
    bank = isr.isr_noise_bank(sigma, 12345, 7, 0, count, d)
    n = count * d
    x = bank.to(torch.float64)
    mean, var = float(x.mean()), float(x.var(unbiased=False))
    assert abs(mean) < 5 * sigma / np.sqrt(n)
    assert abs(var / sigma ** 2 - 1) < 5 * np.sqrt(2.0 / n) + 1e-9      # the discrete law's variance is sigma^2 to < 1e-13 for sigma >= 2
    mp.mp.dps = 50
    K = 12 * sigma
    w = [mp.e ** (-(mp.mpf(k) ** 2) / (2 * mp.mpf(sigma) ** 2)) for k in range(0, K + 1)]
    Z = w[0] + 2 * sum(w[1:])
    pmf = lambda k: w[abs(k)] / Z if abs(k) <= K else mp.mpf(0)
    step = max(1, sigma // 8)
    edges = list(range(-3 * sigma, 3 * sigma + 1, step))                 # cells [e_i, e_{i+1}) plus the two tails
    obs = torch.histc(x, bins=len(edges) - 1, min=edges[0] - 0.5, max=edges[-1] - 0.5).cpu().numpy()
    lo_tail = float((x < edges[0] - 0.5).sum()); hi_tail = float((x > edges[-1] - 0.5).sum())
    obs = np.concatenate([[lo_tail], obs, [hi_tail]])
    probs = [float(sum(pmf(k) for k in range(-K, edges[0])))]
    probs += [float(sum(pmf(k) for k in range(a, b))) for a, b in zip(edges, edges[1:])]
    probs += [float(sum(pmf(k) for k in range(edges[-1], K + 1)))]
    assert abs(sum(probs) - 1) < 1e-12 and int(obs.sum()) == n
    exp = np.array(probs) * n
    chi2 = float(((obs - exp) ** 2 / exp).sum())
    assert chi2 < 110.0, chi2          # 49 degrees of freedom: P[chi2 > 110] ~ 1e-6


# ---- S3-S6: layer tensors ----------------------------------------------------

def _check_all_tensors(isr, blob, x, sigma, seed=3, image=1, phase=1, sample=17, chunk=4, min_fused=0, fusion=1):
    """Every tensor of one noisy copy against the oracle.  With fusion on (the default) a tensor that
    a fused kernel stores is that kernel's own output; a tensor that no fused kernel stores (the
    output of a convolution folded into a residual add, the 112x112 first-layer output under the
    pooling fusion, the middle tensors of a block kernel) is served by the op-by-op kernels, so that
    comparison checks those kernels and not the fused ones -- isr_debug_tensor_source says which.
    The fused kernels are covered by the tensors they do store (block outputs), by the logits of
    this copy below, and by the multi-copy logits check that follows every fused-kernel test.
    min_fused: at least that many tensors must come from fused kernels (guards the test's premise)."""
    m = _load(isr, blob, chunk)
    isr.isr_set_fusion(m, fusion)
    om = oracle.Model(blob)
    a0 = oracle.noisy(x, sigma, seed, image, phase, sample)
    logits, tensors = om.forward(a0)
    n_fused = 0
    for tid in sorted(tensors):
        c, h, w, _ = om.tensor_shape(tid)
        got = isr.isr_debug_tensor(m, x, sigma, seed, image, phase, sample, tid, (c, h, w))
        bad = np.argwhere(got != tensors[tid])
        src = "fused" if isr.isr_debug_tensor_source(m, tid) else "op-by-op"
        n_fused += src == "fused"
        assert bad.size == 0, f"tensor {tid} ({src} plan) shape {(c, h, w)}: {len(bad)} mismatches, first at {bad[0]}"
    assert n_fused >= min_fused, (n_fused, min_fused)
    gl, ga, gc = isr.isr_debug_forward(m, x, sigma, seed, image, phase, sample, 1)
    assert np.array_equal(gl[0], logits)
    m.close()


def test_layer_tensors_tiny(isr):
    _say("layer parity tiny")
    _check_all_tensors(isr, synth.build_model(0), synth.make_image(0, 1), 32)


def test_layer_tensors_resnet20(isr):
    _say("layer parity resnet20")
    _check_all_tensors(isr, synth.build_model(1), synth.make_image(1, 1), 64)


def test_layer_tensors_resnet50_small(isr):
    _say("layer parity resnet50 at 64x64")
    _check_all_tensors(isr, synth.build_model(3, size=64), synth.make_image(3, 1, shape=(3, 64, 64)), 128)


def test_layer_tensors_odd_shapes(isr):
    """Channel counts that are not multiples of 16, 5x5 / 7x7 / 1x1 kernels,
    strides, shifts of 0 and 31, non-trivial zero-points, both add signs."""
    _say("layer parity odd shapes")
    rng = np.random.default_rng(11)
    b = NetBuilder(rng=np.random.default_rng(12), in_shape=(3, 20, 12), num_classes=7)
    t0 = b.tensor(3, 20, 12, 0, 74.0)
    t1 = b.conv(t0, 5, 5, 1, 2, True, sh=rng.integers(6, 10, size=5))
    t2 = b.conv(t1, 40, 3, 2, 1, False, zp_out=9, sh=rng.integers(5, 9, size=40))
    t3 = b.conv(t2, 40, 1, 1, 0, True, sh=rng.integers(4, 8, size=40), zp_out=-100)
    t4 = b.add(t2, t3, False, ma=-600000, mb=900000, sh=20, zp_out=-5)
    t5 = b.conv(t4, 70, 3, 1, 1, True, sh=np.concatenate([[0, 31], rng.integers(5, 9, size=68)]))
    t6 = b.maxpool(t5, 3, 2, 1)
    t7 = b.conv(t6, 130, 1, 2, 0, False, sh=rng.integers(4, 8, size=130))
    t8 = b.conv(t7, 64, 1, 1, 0, True, sh=rng.integers(5, 9, size=64))
    t9 = b.conv(t8, 64, 1, 1, 0, True, sh=rng.integers(5, 9, size=64))   # Cin 64: flat 1x1 path
    t10 = b.maxpool(t9, 2, 1, 0)
    g = b.gap(t10)
    b.fc(g, 7)
    x = np.random.default_rng(5).integers(0, 256, size=(3, 20, 12)).astype(np.uint8)
    _check_all_tensors(isr, b.blob(), x, 64)


def test_first_layer_7x7_stride2(isr):
    _say("layer parity 7x7 stem")
    b = NetBuilder(rng=np.random.default_rng(21), in_shape=(3, 36, 28), num_classes=4)
    t0 = b.tensor(3, 36, 28, 0, 74.0)
    t1 = b.conv(t0, 24, 7, 2, 3, True)
    t2 = b.maxpool(t1, 3, 2, 1)
    b.fc(b.gap(t2), 4)
    x = np.random.default_rng(6).integers(0, 256, size=(3, 36, 28)).astype(np.uint8)
    _check_all_tensors(isr, b.blob(), x, 32)


@pytest.mark.parametrize("shape", [(32, 32), (48, 16), (7, 64)])
def test_first_layer_3x3_into_16_channels(isr, shape):
    """The LDS-resident first layer of the narrow nets (3x3, stride 1, pad 1, 16 stored
    channels): 13 real channels, ReLU off with a non-trivial output zero-point, one variant
    with power-of-two multipliers (rounding ties), 6 copies (ragged against 4 images per
    workgroup); image sizes with one, two and four 16-pixel strips."""
    h, w = shape
    _say(f"layer parity first 3x3 layer {h}x{w}")
    for pow2 in (False, True):
        b = NetBuilder(rng=np.random.default_rng(91), in_shape=(3, h, w), num_classes=4)
        kw = dict(m0=np.full(13, 1 << 30, dtype=np.int64), sh=np.full(13, 7)) if pow2 else {}
        t1 = b.conv(b.tensor(3, h, w, 0, 74.0), 13, 3, 1, 1, pow2, zp_out=-128 if pow2 else 9, **kw)
        t2 = b.conv(t1, 32, 3, 2, 1, True)
        b.fc(b.gap(t2), 4)
        blob = b.blob()
        x = np.random.default_rng(13).integers(0, 256, size=(3, h, w)).astype(np.uint8)
        _check_all_tensors(isr, blob, x, 64, sample=1, chunk=3)
        m = _load(isr, blob, 6)
        om = oracle.Model(blob)
        lg, am, cnt = isr.isr_debug_forward(m, x, 128, 5, 2, 0, 7, 6)
        olg, oam, ocnt = om.mc(x, 128, 5, 2, 0, 7, 6)
        assert np.array_equal(lg, olg) and np.array_equal(cnt, ocnt)
        m.close()


@pytest.mark.parametrize("shape", [(224, 224), (64, 64), (37, 28), (30, 44), (9, 8)])
def test_first_layer_fused_with_max_pooling(isr, shape):
    """7x7/2 convolution into 64 channels followed by 3x3/2 max pooling (one fused kernel):
    every tensor against the oracle, at the full 224 x 224 size, sizes with odd row
    counts, ragged last bands and images narrower than one fragment row."""
    h, w = shape
    _say(f"layer parity fused stem + pool {h}x{w}")
    b = NetBuilder(rng=np.random.default_rng(31), in_shape=(3, h, w), num_classes=5)
    t0 = b.tensor(3, h, w, 0, 74.0)
    t1 = b.conv(t0, 61, 7, 2, 3, True, zp_out=-100)
    t2 = b.maxpool(t1, 3, 2, 1)
    t3 = b.conv(t2, 64, 1, 1, 0, True)
    b.fc(b.gap(t3), 5)
    x = np.random.default_rng(7).integers(0, 256, size=(3, h, w)).astype(np.uint8)
    _check_all_tensors(isr, b.blob(), x, 64, sample=3, chunk=5)


@pytest.mark.parametrize("shape", [(150, 100), (67, 124), (100, 160), (35, 224), (3, 128)])
def test_first_layer_fused_with_max_pooling_in_several_bands(isr, shape):
    """Images of more pooled rows than a workgroup makes, in one strip of columns (16 rows) and in two (8), whose last band and
    last wave are partly or wholly outside the image."""
    test_first_layer_fused_with_max_pooling(isr, shape)


def test_identity_residual_blocks_in_one_kernel(isr):
    """conv3x3 -> conv3x3 -> add with the block input, at the three shapes that run as one
    LDS-resident kernel (16 channels at 32x32, 32 at 16x16, 64 at 8x8): non-trivial zero-points
    on every tensor, ReLU on and off, power-of-two multipliers (rounding ties) in one block,
    7 copies (ragged against 2 and 4 images per workgroup)."""
    _say("layer parity fused identity blocks")
    rng = np.random.default_rng(71)
    b = NetBuilder(rng=np.random.default_rng(72), in_shape=(3, 32, 32), num_classes=6)
    t = b.conv(b.tensor(3, 32, 32, 0, 74.0), 16, 3, 1, 1, True)
    def block(t, ch, relu1, relu_out, z1, z2, zo, pow2=False):
        m0 = np.full(ch, 1 << 30, dtype=np.int64) if pow2 else None
        u = b.conv(t, ch, 3, 1, 1, relu1, zp_out=z1, m0=m0, sh=np.full(ch, 9) if pow2 else None)
        u = b.conv(u, ch, 3, 1, 1, False, zp_out=z2)
        if pow2:
            return b.add(t, u, relu_out, ma=1 << 19, mb=1 << 19, sh=20, zp_out=zo)
        return b.add(t, u, relu_out, zp_out=zo)
    t = block(t, 16, True, True, -128, 0, -128)
    t = block(t, 16, False, False, 7, -5, 3)
    t = block(t, 16, True, True, -100, 9, -120, pow2=True)
    t = b.conv(t, 32, 3, 2, 1, True)
    t = block(t, 32, True, False, -128, 4, -2)
    t = block(t, 32, False, True, 11, 0, -128, pow2=True)
    t = b.conv(t, 64, 3, 2, 1, True)
    t = block(t, 64, True, True, -128, 0, -128)
    t = block(t, 64, False, False, -9, 13, 6)
    b.fc(b.gap(t), 6)
    blob = b.blob()
    x = np.random.default_rng(11).integers(0, 256, size=(3, 32, 32)).astype(np.uint8)
    _check_all_tensors(isr, blob, x, 64, sample=4, chunk=3)
    m = _load(isr, blob, 7)
    om = oracle.Model(blob)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 100, 7)
    olg, oam, ocnt = om.mc(x, 64, 2, 1, 1, 100, 7)
    assert np.array_equal(lg, olg) and np.array_equal(cnt, ocnt)
    m.close()


def test_downsampling_residual_blocks_in_one_kernel(isr):
    """conv3x3 stride 2 -> conv3x3 with a 1x1 stride-2 projection shortcut and the add, at
    the two shapes that run as one LDS-resident kernel (16 -> 32 channels at 32x32 -> 16x16,
    32 -> 64 at 16x16 -> 8x8): zero-points on every tensor, ReLU on and off, a variant with
    power-of-two multipliers (rounding ties), 5 copies (ragged against 2 images per workgroup)."""
    _say("layer parity fused down-sampling blocks")
    for pow2 in (False, True):
        b = NetBuilder(rng=np.random.default_rng(101), in_shape=(3, 32, 32), num_classes=6)
        t = b.conv(b.tensor(3, 32, 32, 0, 74.0), 16, 3, 1, 1, True, zp_out=-128 if not pow2 else -90)
        def down(x, ch, z1, z2, zp, zo, relu1, relu_out):
            kw = dict(m0=np.full(ch, 1 << 30, dtype=np.int64), sh=np.full(ch, 8)) if pow2 else {}
            u = b.conv(x, ch, 3, 2, 1, relu1, zp_out=z1, **kw)
            u = b.conv(u, ch, 3, 1, 1, False, zp_out=z2, **kw)
            r = b.conv(x, ch, 1, 2, 0, False, zp_out=zp)
            if pow2:
                return b.add(u, r, relu_out, ma=1 << 19, mb=1 << 19, sh=20, zp_out=zo)
            return b.add(u, r, relu_out, zp_out=zo)
        t = down(t, 32, -128, 0, 0, -128, True, True)
        t = down(t, 64, 11, -7, 5, 3, False, False)
        b.fc(b.gap(t), 6)
        blob = b.blob()
        x = np.random.default_rng(14).integers(0, 256, size=(3, 32, 32)).astype(np.uint8)
        _check_all_tensors(isr, blob, x, 64, sample=3, chunk=3)
        m = _load(isr, blob, 5)
        om = oracle.Model(blob)
        lg, am, cnt = isr.isr_debug_forward(m, x, 32, 6, 1, 1, 40, 5)
        olg, oam, ocnt = om.mc(x, 32, 6, 1, 1, 40, 5)
        assert np.array_equal(lg, olg) and np.array_equal(cnt, ocnt)
        m.close()


@pytest.mark.parametrize("copies", [1, 3, 256, 257, 1025])
@pytest.mark.parametrize("net", ["stages", "down"])
def test_stages_of_the_nets_on_32x32_images(isr, net, copies):
    """One launch per stage: first layer + blocks + down-sampling, a stage without blocks, blocks + pooling + fully
    connected layer with more classes than a wave has lanes; constants in the top-byte form, with ties, and in the
    general form; one and several images per workgroup with ragged last ones; single votes and batched ones."""
    _say(f"narrow stages {net} {copies}")
    b = NetBuilder(rng=np.random.default_rng(91), in_shape=(3, 32, 32), num_classes=70)
    t = b.conv(b.tensor(3, 32, 32, 0, 74.0), 16, 3, 1, 1, True)
    def block(t, ch, zo=-128, **kw):
        u = b.conv(t, ch, 3, 1, 1, True, **({"m0": np.full(ch, 1 << 30, dtype=np.int64)} if "ma" in kw else {}))
        return b.add(t, b.conv(u, ch, 3, 1, 1, False), True, zp_out=zo, **kw)
    def down(t, ch):
        u = b.conv(b.conv(t, ch, 3, 2, 1, True), ch, 3, 1, 1, False)
        return b.add(b.conv(t, ch, 1, 2, 0, False), u, True)
    if net == "stages":
        t = block(t, 16)
        t = block(t, 16, ma=1 << 19, mb=1 << 19, sh=20)        # exact halves in the first convolution and in the add
        t = down(block(t, 16, zo=-100), 32)                    # general form; another zero-point in the border of x
        t = down(t, 64)
        t = block(block(block(t, 64), 64, zo=-90), 64)
    else:
        t = b.conv(t, 32, 3, 2, 1, True)
    b.fc(b.gap(t), 70)
    blob = b.blob()
    m = _load(isr, blob, copies)
    om = oracle.Model(blob)
    x = np.random.default_rng(12).integers(0, 256, size=(3, 32, 32)).astype(np.uint8)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 100, copies)
    k = min(copies, 5)
    olg, oam, _ = om.mc(x, 64, 2, 1, 1, 100 + copies - k, k)
    assert np.array_equal(lg[-k:], olg) and np.array_equal(am[-k:], oam)
    assert np.array_equal(cnt, np.bincount(am, minlength=70))
    isr.isr_set_fusion(m, 0)
    lg0, am0, cnt0 = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 100, copies)
    assert np.array_equal(lg, lg0) and np.array_equal(am, am0) and np.array_equal(cnt, cnt0)
    votes = []
    for fusion in (0, 1):
        isr.isr_set_fusion(m, fusion)
        votes.append(isr.isr_predict_batch(m, np.stack([x, 255 - x]), [(0, 64, 1), (1, 32, 2), (0, 32, 3)], copies, ALPHA, seed=5)[1])
    assert np.array_equal(votes[0], votes[1]) and (votes[0].sum(axis=1) == copies).all()
    m.close()


@pytest.mark.parametrize("channels", [1, 2, 3])
def test_noise_of_few_copies_is_drawn_by_channel(isr, channels):
    """Eight waves an image draw a channel of a quad of pixels at a time: images of one to three channels, few copies (eight
    waves) and many (four), blocks whose descriptors are fetched ahead in every stage."""
    _say(f"narrow stages of {channels}-channel images")
    b = NetBuilder(rng=np.random.default_rng(92), in_shape=(channels, 32, 32), num_classes=7)
    t = b.conv(b.tensor(channels, 32, 32, 0, 74.0), 16, 3, 1, 1, True)
    for ch in (16, 32, 64):
        if ch > 16:
            u = b.conv(b.conv(t, ch, 3, 2, 1, True), ch, 3, 1, 1, False)
            t = b.add(b.conv(t, ch, 1, 2, 0, False), u, True)
        for zo in (-128, -70, -128):
            t = b.add(t, b.conv(b.conv(t, ch, 3, 1, 1, True), ch, 3, 1, 1, False), True, zp_out=zo)
    b.fc(b.gap(t), 7)
    blob = b.blob()
    om = oracle.Model(blob)
    x = np.random.default_rng(13).integers(0, 256, size=(channels, 32, 32)).astype(np.uint8)
    olg, oam, _ = om.mc(x, 64, 2, 1, 1, 100, 4)
    m = _load(isr, blob, 300)
    for copies in (4, 300):
        lg, am, _ = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 100, copies)
        assert np.array_equal(lg[:4], olg) and np.array_equal(am[:4], oam), copies
    m.close()


@pytest.mark.parametrize("copies", [1, 256, 257])
@pytest.mark.parametrize("blocks", [(0, 0, 0), (1, 0, 2), (0, 3, 1), (2, 1, 0)])
def test_three_stages_of_few_copies_in_one_launch(isr, blocks, copies):
    """Nets on 32x32 images whose stages run in one launch up to 256 copies and in three beyond, with no and several identity blocks a
    stage: logits against the oracle, all copies against the op-by-op kernels, and which launch it was."""
    _say(f"narrow stages of {blocks} blocks, {copies} copies")
    b = NetBuilder(rng=np.random.default_rng(93), in_shape=(3, 32, 32), num_classes=7)
    t = b.conv(b.tensor(3, 32, 32, 0, 74.0), 16, 3, 1, 1, True)
    for ch, n in zip((16, 32, 64), blocks):
        if ch > 16:
            u = b.conv(b.conv(t, ch, 3, 2, 1, True), ch, 3, 1, 1, False)
            t = b.add(b.conv(t, ch, 1, 2, 0, False), u, True)
        for i in range(n):
            t = b.add(t, b.conv(b.conv(t, ch, 3, 1, 1, True), ch, 3, 1, 1, False), True, zp_out=-128 + 30 * i)
    b.fc(b.gap(t), 7)
    blob = b.blob()
    om = oracle.Model(blob)
    x = np.random.default_rng(13).integers(0, 256, size=(3, 32, 32)).astype(np.uint8)
    n = min(copies, 4)
    olg, oam, _ = om.mc(x, 64, 2, 1, 1, 100, n)
    m = _load(isr, blob, 300)
    isr.isr_profile(m, 1)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 100, copies)
    names = [k["name"] for k in isr.isr_profile_read(m)]
    whole = blocks[2] > 0          # without blocks the last stage has no kernel of its own
    assert ("narrow_chain_kernel" in names) == (whole and copies <= 256), names
    assert np.array_equal(lg[:n], olg) and np.array_equal(am[:n], oam)
    isr.isr_set_fusion(m, 0)
    plain = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 100, copies)
    assert np.array_equal(lg, plain[0]) and np.array_equal(am, plain[1]) and np.array_equal(cnt, plain[2])
    m.close()


@pytest.mark.parametrize("first", ["16 channels", "7x7 and pooling", "noise launch"])
def test_both_phases_of_a_certification_in_one_list(isr, first):
    """Chunks and launches that end inside either phase and inside a pair: tallies against those of the phases alone, for first
    layers that draw their own noise and for the noise launch, single calls and batches, and the rounded continuous noise."""
    _say(f"phases in one list: {first}")
    b = NetBuilder(rng=np.random.default_rng(17), in_shape=(3, 32, 32), num_classes=9)
    t = b.tensor(3, 32, 32, 0, 74.0)
    if first == "16 channels":
        t = b.conv(t, 16, 3, 1, 1, True)
        t = b.add(t, b.conv(b.conv(t, 16, 3, 1, 1, True), 16, 3, 1, 1, False), True)
    else:
        t = b.maxpool(b.conv(t, 64, 7, 2, 3, True), 3, 2, 1)
    b.fc(b.gap(t), 9)
    m = _load(isr, b.blob(), 7)
    isr.isr_set_fusion(m, 0 if first == "noise launch" else 1)
    x = np.random.default_rng(18).integers(0, 256, size=(3, 32, 32)).astype(np.uint8)
    tally = lambda img, sigma, image_id, phase, n: isr.isr_debug_forward(m, img, sigma, 3, image_id, phase, 0, n)[2]
    for n0, n in ((5, 16), (7, 7), (23, 1)):
        _, c0, c1 = isr.isr_certify(m, x, 48, n0, n, ALPHA, seed=3, image_id=6)
        assert np.array_equal(c0, tally(x, 48, 6, 0, n0)) and np.array_equal(c1, tally(x, 48, 6, 1, n))
        _, c = isr.isr_predict(m, x, 48, n0, ALPHA, seed=3, image_id=6)
        assert np.array_equal(c, c0)
        items = [(0, 48, 1), (1, 90, 2), (0, 90, 3)]
        _, c0, c1 = isr.isr_certify_batch(m, np.stack([x, 255 - x]), items, n0, n, ALPHA, seed=3)
        for i, (im, sigma, image_id) in enumerate(items):
            img = 255 - x if im else x
            assert np.array_equal(c0[i], tally(img, sigma, image_id, 0, n0)) and np.array_equal(c1[i], tally(img, sigma, image_id, 1, n))
        _, q0, q1 = isr.isr_float_certify(m, x, 48.0, n0, n, ALPHA, isr.FLOATRS_QUANT, seed=3, image_id=6)
        for phase, k, q in ((0, n0, q0), (1, n, q1)):
            assert np.array_equal(q, isr.isr_float_debug_forward(m, x, 48.0, 3, 6, phase, 0, k, isr.FLOATRS_QUANT)[2])
    m.close()


@pytest.mark.parametrize("shape", [(30, 20), (28, 28), (5, 40)])
def test_bottleneck_blocks_in_one_kernel(isr, shape):
    """conv1x1 -> conv3x3 (64 middle channels) [-> conv1x1 + add with the block input] as one
    kernel working on 14 x 14 pixel tiles: images that leave ragged tiles in both directions,
    one exactly two tiles wide and one lower than a tile; block widths 64 / 128 / 256 (one to
    four K steps); zero-points on every tensor, ReLU on and off, a block with power-of-two
    multipliers (rounding ties), a block whose residual comes from a projection (head only)."""
    h, w = shape
    _say(f"layer parity fused bottleneck blocks {h}x{w}")
    b = NetBuilder(rng=np.random.default_rng(81), in_shape=(3, h, w), num_classes=5)
    t = b.conv(b.tensor(3, h, w, 0, 74.0), 64, 3, 1, 1, True)
    def block(x, cx, z1, z2, z3, zo, relu12=True, relu_out=True, pow2=False, project=False):
        kw = dict(m0=np.full(64, 1 << 30, dtype=np.int64), sh=np.full(64, 9)) if pow2 else {}
        u = b.conv(x, 64, 1, 1, 0, relu12, zp_out=z1, **kw)
        u = b.conv(u, 64, 3, 1, 1, relu12, zp_out=z2, **kw)
        if project:
            r = b.conv(x, cx, 1, 1, 0, False, zp_out=5)
            u = b.conv(u, cx, 1, 1, 0, False, zp_out=z3)
            return b.add(r, u, relu_out, zp_out=zo)
        u = b.conv(u, cx, 1, 1, 0, False, zp_out=z3)
        if pow2:
            return b.add(x, u, relu_out, ma=1 << 19, mb=1 << 19, sh=20, zp_out=zo)
        return b.add(x, u, relu_out, zp_out=zo)
    t = block(t, 64, -128, -128, 0, -128)
    t = block(t, 256, -100, 7, 3, -128, project=True)
    t = block(t, 256, -128, -128, 0, -128)
    t = block(t, 256, 9, -20, -6, 11, relu12=False, relu_out=False)
    t = block(t, 256, -128, -128, 4, -128, pow2=True)
    t = b.conv(t, 128, 1, 1, 0, True)
    t = block(t, 128, -128, -90, 0, -128)
    b.fc(b.gap(t), 5)
    blob = b.blob()
    x = np.random.default_rng(12).integers(0, 256, size=(3, h, w)).astype(np.uint8)
    _check_all_tensors(isr, blob, x, 64, sample=2, chunk=3)
    m = _load(isr, blob, 5)
    om = oracle.Model(blob)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 3, 1, 1, 50, 5)
    olg, oam, ocnt = om.mc(x, 64, 3, 1, 1, 50, 5)
    assert np.array_equal(lg, olg) and np.array_equal(cnt, ocnt)
    m.close()


@pytest.mark.parametrize("shape,copies,layers,kernels", [
    ((8, 28), 1793, None, (2, 1)),          # one tile an image, 256 workgroups with seven of them, one with an eighth
    ((9, 32), 448, None, (2, 1)),           # four tiles an image, three of them nearly outside; seven tiles each
    ((9, 32), 320, None, (2, 0)),           # five tiles each: identity blocks only
    ((8, 28), 1279, None, (0, 0)), ((8, 28), 1535, None, (2, 0)),
    # first blocks in the top-byte form from sixteen rounds of 256 tiles on, the others earlier
    ((5, 40), 1281, "_ByChannel", (2, 0)), ((5, 40), 2047, "_HalvesByChannel", (2, 0)),
    ((5, 40), 2049, "_ByChannel", (2, 1)), ((9, 32), 1025, "_TopForm", (2, 1)), ((9, 32), 1025, "_HalvesInAdds", (2, 1)), ((5, 40), 2048, "_HalvesByChannel", (2, 1)),
    ((8, 28), 1279, "_Clamped", (0, 0)), ((8, 28), 1281, "_Clamped", (2, 0)), ((9, 32), 385, "_Clamped", (2, 1)), ((8, 28), 2560, "_Clamped", (2, 1)),
    # exact halves in the convolutions, next to clamps of -128 and others
    ((8, 28), 1281, "_HalvesInBoth", (0, 0)), ((9, 32), 385, "_HalvesInBoth", (2, 0)), ((5, 40), 1153, "_HalvesInBoth", (2, 1)),
    ((8, 28), 1281, "_HalvesInBothClamped", (2, 0)), ((5, 40), 769, "_HalvesInBothClamped", (2, 1))])
def test_bottleneck_blocks_in_resident_workgroups(isr, builder, shape, copies, layers, kernels):
    """Blocks of 256 channels in launches of many tiles, in each form of the requantisation, on images that leave tiles ragged in both
    directions: against one kernel per op, and two copies against the oracle.  Logits that depend on every pixel."""
    h, w = shape
    _say(f"resident bottleneck blocks {h}x{w}, {copies} copies, {layers}")
    if layers:
        builder(globals()[layers])
    b = NetBuilder(rng=np.random.default_rng(85), in_shape=(3, h, w), num_classes=6)
    t = b.conv(b.tensor(3, h, w, 0, 74.0), 64, 3, 1, 1, True)
    u = b.conv(b.conv(t, 64, 1, 1, 0, False, zp_out=-100), 64, 3, 1, 1, True)
    r = b.conv(t, 256, 1, 1, 0, False, zp_out=5)
    t = b.add(r, b.conv(u, 256, 1, 1, 0, False, zp_out=3), True)
    for k in range(2):
        u = b.conv(b.conv(t, 64, 1, 1, 0, True), 64, 3, 1, 1, False, zp_out=-20 * k)
        t = b.add(t, b.conv(u, 256, 1, 1, 0, False, zp_out=k), k == 1)
    b.fc(b.conv(t, 16, 1, 1, 0, True), 6)
    m = _load(isr, b.blob(), copies)
    x = np.random.default_rng(86).integers(0, 256, size=(3, h, w)).astype(np.uint8)
    isr.isr_profile(m, 1)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 3, copies)
    names = {s["name"]: s["launches"] for s in isr.isr_profile_read(m)}
    assert (names.get("bottleneck_stream_kernel<block>", 0), names.get("bottleneck_stream_kernel<block + projection>", 0)) == kernels, names
    isr.isr_set_fusion(m, 0)
    lg0, am0, cnt0 = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 3, copies)
    m.close()
    assert np.array_equal(lg, lg0) and np.array_equal(am, am0) and np.array_equal(cnt, cnt0)
    assert np.array_equal(lg[:2], oracle.Model(b.blob()).mc(x, 64, 2, 1, 1, 3, 2)[0])


@pytest.mark.parametrize("cin", [192, 256, 320, 512])
def test_bottleneck_heads_of_three_to_eight_k_steps(isr, cin):
    """The opening 1x1 and the 3x3 convolution (64 middle channels) in one kernel for wider inputs than a block's own: more K
    steps than operand stages, against the oracle."""
    _say(f"bottleneck head {cin} input channels")
    b = NetBuilder(rng=np.random.default_rng(83), in_shape=(3, 10, 32), num_classes=5)
    t = b.conv(b.tensor(3, 10, 32, 0, 74.0), cin, 3, 1, 1, True)
    u = b.conv(b.conv(t, 64, 1, 1, 0, True, zp_out=-90), 64, 3, 1, 1, True, zp_out=7)
    u = b.conv(u, 256, 1, 1, 0, False)
    b.fc(b.gap(b.add(b.conv(t, 256, 1, 1, 0, False), u, True)), 5)
    blob = b.blob()
    x = np.random.default_rng(12).integers(0, 256, size=(3, 10, 32)).astype(np.uint8)
    _check_all_tensors(isr, blob, x, 64, sample=2, chunk=3)
    m = _load(isr, blob, 5)
    lg, _, cnt = isr.isr_debug_forward(m, x, 64, 3, 1, 1, 50, 5)
    olg, _, ocnt = oracle.Model(blob).mc(x, 64, 3, 1, 1, 50, 5)
    assert np.array_equal(lg, olg) and np.array_equal(cnt, ocnt)
    m.close()


@pytest.mark.parametrize("shape", [(30, 20), (28, 28), (5, 40)])
def test_bottleneck_blocks_with_128_middle_channels_in_one_kernel(isr, shape):
    """conv1x1 -> conv3x3 (128 middle channels) -> conv1x1 + add with the block input as one kernel on
    14 x 14 pixel tiles: images with ragged tiles in both directions, one exactly two tiles wide, one
    lower than a tile; block widths 512 / 256 / 192 (eight, four and three K steps; 192 leaves the
    last round of output-channel passes to two of the four waves); zero-points on every tensor, ReLU
    on and off, a block with power-of-two multipliers (rounding ties)."""
    h, w = shape
    _say(f"layer parity fused bottleneck blocks, 128 middle channels, {h}x{w}")
    b = NetBuilder(rng=np.random.default_rng(83), in_shape=(3, h, w), num_classes=5)
    t = b.conv(b.tensor(3, h, w, 0, 74.0), 64, 3, 1, 1, True)
    t = b.conv(t, 512, 1, 1, 0, True)
    def block(x, cx, z1, z2, z3, zo, relu12=True, relu_out=True, pow2=False):
        kw = dict(m0=np.full(128, 1 << 30, dtype=np.int64), sh=np.full(128, 9)) if pow2 else {}
        u = b.conv(x, 128, 1, 1, 0, relu12, zp_out=z1, **kw)
        u = b.conv(u, 128, 3, 1, 1, relu12, zp_out=z2, **kw)
        u = b.conv(u, cx, 1, 1, 0, False, zp_out=z3)
        if pow2:
            return b.add(x, u, relu_out, ma=1 << 19, mb=1 << 19, sh=20, zp_out=zo)
        return b.add(x, u, relu_out, zp_out=zo)
    t = block(t, 512, -128, -128, 0, -128)
    t = block(t, 512, 9, -20, -6, 11, relu12=False, relu_out=False)
    t = block(t, 512, -128, -128, 4, -128, pow2=True)
    t = b.conv(t, 256, 1, 1, 0, True)
    t = block(t, 256, -100, 7, 3, -128)
    t = b.conv(t, 192, 1, 1, 0, True)
    t = block(t, 192, -128, -90, 0, -128)
    b.fc(b.gap(t), 5)
    blob = b.blob()
    x = np.random.default_rng(15).integers(0, 256, size=(3, h, w)).astype(np.uint8)
    _check_all_tensors(isr, blob, x, 64, sample=2, chunk=3, min_fused=5, fusion=2)
    m = _load(isr, blob, 5)
    isr.isr_set_fusion(m, 2)
    om = oracle.Model(blob)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 3, 1, 1, 50, 5)
    olg, oam, ocnt = om.mc(x, 64, 3, 1, 1, 50, 5)
    assert np.array_equal(lg, olg) and np.array_equal(cnt, ocnt)
    isr.isr_set_fusion(m, False)
    lg2, _, _ = isr.isr_debug_forward(m, x, 64, 3, 1, 1, 50, 5)
    assert np.array_equal(lg2, olg)
    m.close()


def test_residual_computed_by_a_second_convolution(isr):
    """Projection-shortcut pattern: the residual of an add is the output of a 1x1
    convolution issued right before the add's other convolution; the fused plan then
    computes both in one kernel and never stores the residual.  Main convolution 3x3
    (gather), 1x1 stride 2 (gather) and 1x1 stride 1 (plain GEMM); channel counts that
    leave a ragged last M tile; K of the two convolutions different; 29 copies."""
    _say("layer parity dual-convolution residual add")
    rng = np.random.default_rng(61)
    b = NetBuilder(rng=np.random.default_rng(62), in_shape=(3, 12, 12), num_classes=8)
    t0 = b.tensor(3, 12, 12, 0, 74.0)
    t1 = b.conv(t0, 64, 3, 1, 1, True)
    t2 = b.conv(t1, 192, 1, 1, 0, False, zp_out=11)          # residual producer (K = 64)
    t3 = b.conv(t1, 192, 3, 1, 1, False, zp_out=-9)          # main, K = 576
    t4 = b.add(t2, t3, True)
    u = b.conv(t4, 128, 3, 2, 1, True)                       # 6 x 6
    r = b.conv(u, 320, 1, 1, 0, False)                       # residual producer (K = 128)
    mn = b.conv(t4, 320, 1, 2, 0, False)                     # main: 1x1 stride 2, K = 192
    t5 = b.add(mn, r, True)                                  # residual is the second operand here
    r2 = b.conv(t5, 64, 1, 1, 0, False)                      # 64 output channels: the 64 x 256 tile
    m2 = b.conv(t5, 64, 1, 1, 0, True)
    t6 = b.add(r2, m2, False, ma=-500000, mb=800000, sh=20)
    b.fc(b.gap(t6), 8)
    blob = b.blob()
    x = np.random.default_rng(10).integers(0, 256, size=(3, 12, 12)).astype(np.uint8)
    _check_all_tensors(isr, blob, x, 64, sample=1, chunk=3)
    m = _load(isr, blob, 29)
    om = oracle.Model(blob)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 1, 1, 1, 0, 29)
    olg, oam, ocnt = om.mc(x, 64, 1, 1, 1, 0, 29)
    assert np.array_equal(lg, olg) and np.array_equal(cnt, ocnt)
    isr.isr_set_fusion(m, False)
    lg2, _, _ = isr.isr_debug_forward(m, x, 64, 1, 1, 1, 0, 29)
    assert np.array_equal(lg2, olg)
    m.close()


@pytest.mark.parametrize("copies,one_shift,wide", [(975, True, 0), (983, True, 2), (1047, True, 0), (1967, True, 1), (2211, True, 2), (983, False, 0)])
def test_convolution_pairs_in_launches_of_many_tiles(isr, builder, copies, one_shift, wide):
    """Pairs of 256 channels a workgroup from 768 tiles of 128 pixels on, where results come in pairs and the last 256 tiles leave few CUs idle
    (4 and 17 K steps, 768, 820, 1540 and 1728 tiles); the last tile ragged.  A main
    convolution of stride 2 and one that is a plain GEMM, K steps of both unequal: against one kernel per op, and two copies against the oracle."""
    _say(f"convolution pairs, {copies} copies, {one_shift}, {wide}")
    if not one_shift:
        builder(_ByChannel)
    b = NetBuilder(rng=np.random.default_rng(66), in_shape=(3, 20, 20), num_classes=8)
    ta = b.conv(b.tensor(3, 20, 20, 0, 74.0), 64, 3, 2, 1, True)
    u = b.conv(b.conv(ta, 128, 1, 1, 0, True), 192, 3, 2, 1, True)
    r = b.conv(u, 1024, 1, 1, 0, False)                                       # the residual, K = 192
    t = b.add(b.conv(ta, 1024, 1, 2, 0, False, zp_out=-9), r, True)           # main: stride 2, K = 64
    u = b.conv(t, 64, 1, 1, 0, True)
    r = b.conv(t, 1024, 1, 1, 0, False, zp_out=5)                             # K = 1024
    t = b.add(r, b.conv(u, 1024, 1, 1, 0, False), False)                      # main: K = 64
    b.fc(b.conv(t, 16, 1, 1, 0, True), 8)
    m = _load(isr, b.blob(), copies)
    x = np.random.default_rng(67).integers(0, 256, size=(3, 20, 20)).astype(np.uint8)
    isr.isr_profile(m, 1)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 3, copies)
    pairs = {s["name"]: s["launches"] for s in isr.isr_profile_read(m) if ", 64, 2, 2, " in s["name"]}
    assert sum(pairs.values()) == 2 and sum(n for name, n in pairs.items() if "<256, 128, " in name) == wide, pairs
    isr.isr_set_fusion(m, 0)
    lg0, am0, cnt0 = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 3, copies)
    m.close()
    assert np.array_equal(lg, lg0) and np.array_equal(am, am0) and np.array_equal(cnt, cnt0)
    assert np.array_equal(lg[:2], oracle.Model(b.blob()).mc(x, 64, 2, 1, 1, 3, 2)[0])


def test_exact_halves_in_both_requantisations(isr):
    """Power-of-two multipliers make acc * M0 and the residual sum land on exact halves
    all the time (negative ones included), so the rounding's sign correction decides
    results: layers that cannot take the tie-free shortcut, next to ones that can."""
    _say("layer parity with rounding ties")
    rng = np.random.default_rng(41)
    b = NetBuilder(rng=np.random.default_rng(42), in_shape=(3, 16, 16), num_classes=6)
    t0 = b.tensor(3, 16, 16, 0, 74.0)
    m_pow2 = np.full(64, 1 << 30, dtype=np.int64)
    m_mixed = np.where(np.arange(64) % 2 == 0, 1 << 30, (1 << 30) + 12345).astype(np.int64)
    t1 = b.conv(t0, 64, 3, 1, 1, True, m0=m_pow2, sh=np.full(64, 9))
    t2 = b.conv(t1, 64, 3, 1, 1, False, m0=m_mixed, sh=np.full(64, 10), zp_out=3)
    t3 = b.conv(t2, 64, 1, 1, 0, False, m0=m_pow2, sh=np.full(64, 8), zp_out=-7)
    t4 = b.add(t2, t3, True, ma=1 << 19, mb=1 << 19, sh=20, zp_out=-20)      # ties in the fused add
    t5 = b.conv(t4, 128, 1, 1, 0, False, sh=rng.integers(6, 9, size=128))
    t6 = b.conv(t5, 128, 3, 1, 1, False, m0=np.full(128, 3 << 29, dtype=np.int64), sh=np.full(128, 9))
    t7 = b.add(t5, t6, False, ma=700001, mb=-(1 << 20), sh=20, zp_out=5)
    b.fc(b.gap(t7), 6)
    x = np.random.default_rng(8).integers(0, 256, size=(3, 16, 16)).astype(np.uint8)
    _check_all_tensors(isr, b.blob(), x, 64, sample=2, chunk=3)


@pytest.mark.parametrize("sh,m0,zp,relu_a,ma,mb,add_sh", [
    (3, (1 << 31) - 1, -128, True, (1 << 20) - 1, (1 << 20) - 3, 20),     # smallest shift of the top-byte form: nearly every output saturates
    (9, None, 0, True, 700001, 800003, 20),                               # identity block: a rectified and a signed operand
    (9, None, 5, False, 900001, 1000003, 20),                             # two signed operands: the sum leaves int32 and saturates
    (10, None, -128, False, -900001, 1000003, 20),                        # a negative multiplier
    (9, None, 127, False, (1 << 23) - 1, (1 << 22) + 1, 23),              # largest shift of the add in the top-byte form
    (8, None, -3, True, 5, 3, 2),                                         # small multipliers and shift
    (22, (1 << 31) - 1, 0, False, 700001, 800003, 20),                    # largest shift: every output at its zero point
    (9, 3 << 29, 0, True, 700001, 800003, 20),                            # convolution with exact halves
    (2, None, 0, True, 700001, 800003, 20),                               # shift below the top-byte form
    (9, None, 0, True, (1 << 20) + 7, 800003, 20),                        # add multiplier above it
])
def test_forms_of_the_requantisation(isr, sh, m0, zp, relu_a, ma, mb, add_sh):
    """Every form of the epilogue (value or top byte, with and without ties, narrow and wide add) at the ends of its
    range, in the direct-to-LDS kernel (plain, fused add, dual convolution) and the bottleneck kernel."""
    _say(f"requantisation forms {sh} {m0} {zp} {relu_a} {ma} {mb} {add_sh}")
    _check_forms(isr, lambda c: np.full(c, sh), m0, zp, relu_a, ma, mb, add_sh)


@pytest.mark.parametrize("sh,by_channel,m0,zp,relu_a,ma,mb,add_sh", [
    (9, True, None, 0, True, 700001, 800003, 20),                    # shifts that differ: the top-byte form, narrow and wide add
    (9, True, None, 5, False, 900001, 1000003, 20),
    (3, True, (1 << 31) - 1, -128, True, (1 << 20) - 1, (1 << 20) - 3, 20),
    (2, False, (1 << 31) - 1, 0, True, 3, 1, 1),                     # one shift, pairs of results: the ends of the shifts
    (2, False, None, 127, False, (1 << 22) - 1, (1 << 21) + 1, 24),
    (22, False, (1 << 31) - 1, -128, False, (1 << 22) + 1, -(1 << 21) - 1, 23),
    (5, False, None, 3, True, 40000001 >> 4, 3, 22),                 # high words beyond 24 bits
])
def test_forms_of_the_requantisation_by_the_layers_shifts(isr, sh, by_channel, m0, zp, relu_a, ma, mb, add_sh):
    """Layers whose channels share one shift take results in pairs; those whose shifts differ keep the other forms."""
    _say(f"requantisation forms by shift {sh} {by_channel} {m0} {zp} {relu_a} {ma} {mb} {add_sh}")
    _check_forms(isr, lambda c: sh + (np.arange(c) % 3 if by_channel else np.zeros(c, dtype=np.int64)), m0, zp, relu_a, ma, mb, add_sh)


def _check_forms(isr, shifts, m0, zp, relu_a, ma, mb, add_sh):
    b = NetBuilder(rng=np.random.default_rng(71), in_shape=(3, 9, 12), num_classes=5)
    kw = lambda c: dict(sh=shifts(c), m0=None if m0 is None else np.full(c, m0, dtype=np.int64))
    t0 = b.tensor(3, 9, 12, 0, 74.0)
    t1 = b.conv(t0, 64, 3, 1, 1, relu_a, sh=np.full(64, 8))
    u = b.conv(t1, 64, 1, 1, 0, True, **kw(64))
    u = b.conv(u, 64, 3, 1, 1, True, **kw(64))
    u = b.conv(u, 64, 1, 1, 0, False, zp_out=zp, **kw(64))
    t2 = b.add(t1, u, True, ma=ma, mb=mb, sh=add_sh)           # identity bottleneck block
    s_ = b.conv(t2, 256, 1, 1, 0, False, zp_out=zp, **kw(256))
    u = b.conv(t2, 64, 1, 1, 0, True, **kw(64))
    u = b.conv(u, 64, 3, 1, 1, True, **kw(64))
    u = b.conv(u, 256, 1, 1, 0, False, **kw(256))
    t3 = b.add(s_, u, False, ma=ma, mb=mb, sh=add_sh, zp_out=-128)   # projection bottleneck block
    u = b.conv(t3, 128, 3, 1, 1, False, zp_out=zp, **kw(128))
    v = b.conv(u, 128, 3, 1, 1, relu_a, **kw(128))
    t4 = b.add(v, u, True, ma=ma, mb=mb, sh=add_sh)            # residual add in a convolution's epilogue
    s_ = b.conv(t4, 192, 1, 1, 0, False, zp_out=zp, **kw(192))
    u = b.conv(t4, 192, 3, 1, 1, False, **kw(192))
    t5 = b.add(u, s_, True, ma=ma, mb=mb, sh=add_sh)           # the residual a second convolution
    b.fc(b.gap(t5), 5)
    x = np.random.default_rng(9).integers(0, 256, size=(3, 9, 12)).astype(np.uint8)
    _check_all_tensors(isr, b.blob(), x, 64, sample=2, chunk=3)


class _ByChannel(NetBuilder):
    """Networks quantised per channel: where a test gives no shifts, they differ from channel to channel."""

    def chosen(self, cout, k):
        return True

    def conv(self, tin, cout, k, stride, pad, relu, sh=None, **kw):
        tout = super().conv(tin, cout, k, stride, pad, relu, sh=sh, **kw)
        if sh is None and self.chosen(cout, k):
            op, payload = self.ops[-1]
            shifts = np.frombuffer(payload[-4 * cout:], dtype="<i4") + np.arange(cout, dtype="<i4") % 3
            self.ops[-1] = (op, payload[:-4 * cout] + shifts.astype("<i4").tobytes())
        return tout


class _TopForm(_ByChannel):
    """The same with lower clamps of -128 throughout: without exact halves every layer takes the top-byte form."""

    def conv(self, tin, cout, k, stride, pad, relu, zp_out=None, **kw):
        return super().conv(tin, cout, k, stride, pad, relu, zp_out=-128 if relu else zp_out, **kw)


class _Clamped(NetBuilder):
    """Rectified layers whose zero point, the lower clamp, is above -128: neither pairs of results nor the top-byte form."""

    def conv(self, tin, cout, k, stride, pad, relu, zp_out=None, **kw):
        return super().conv(tin, cout, k, stride, pad, relu, zp_out=-100 if relu else zp_out, **kw)


class _NextByChannel(_ByChannel):
    """One shift in every layer but the 1x1 convolutions into 128 channels."""

    def chosen(self, cout, k):
        return cout == 128 and k == 1


@pytest.fixture
def builder(monkeypatch):
    return lambda cls: monkeypatch.setattr(sys.modules[__name__], "NetBuilder", cls)


@pytest.mark.parametrize("copies", [3, 257, 1025])
def test_stages_of_nets_quantised_per_channel(isr, builder, copies):
    """The general form of the stage kernels in every layer, with one image a workgroup and with several."""
    builder(_ByChannel)
    test_stages_of_the_nets_on_32x32_images(isr, "stages", copies)


@pytest.mark.parametrize("blocks", [(0, 3, 1), (2, 1, 0)])
def test_three_stages_of_nets_quantised_per_channel(isr, builder, blocks):
    """The general form in the kernel of all stages, and, without blocks in the last, in those of one image a workgroup."""
    builder(_ByChannel)
    test_three_stages_of_few_copies_in_one_launch(isr, blocks, 256)


# Layers whose channels share one shift take results in pairs; the top-byte form, which networks quantised per channel take, in each
# kernel that has it:

@pytest.mark.parametrize("form", ["pairs", "top byte"])
@pytest.mark.parametrize("shape", [(224, 224), (37, 28), (9, 8), (150, 100), (35, 224)])
def test_first_layer_with_pooling_in_the_short_forms(isr, shape, form):
    """Ragged strips and bands, with a lower clamp of -128."""
    h, w = shape
    _say(f"first layer with pooling {h}x{w}, {form}")
    b = (NetBuilder if form == "pairs" else _TopForm)(rng=np.random.default_rng(31), in_shape=(3, h, w), num_classes=5)
    t = b.maxpool(b.conv(b.tensor(3, h, w, 0, 74.0), 61, 7, 2, 3, True), 3, 2, 1)
    b.fc(b.gap(b.conv(t, 64, 1, 1, 0, True)), 5)
    x = np.random.default_rng(7).integers(0, 256, size=(3, h, w)).astype(np.uint8)
    _check_all_tensors(isr, b.blob(), x, 64, sample=3, chunk=5)


@pytest.mark.parametrize("cin", [256, 320])
def test_top_form_in_bottleneck_heads(isr, builder, cin):
    builder(_TopForm)
    test_bottleneck_heads_of_three_to_eight_k_steps(isr, cin)


@pytest.mark.parametrize("shape", [(30, 20), (5, 40)])
def test_top_form_in_bottleneck_blocks(isr, builder, shape):
    builder(_TopForm)
    test_bottleneck_blocks_in_one_kernel(isr, shape)


@pytest.mark.parametrize("layers", [_TopForm, _NextByChannel])
@pytest.mark.parametrize("shape,first,stride", [((32, 56), 2, 2), ((20, 60), 2, 1), ((36, 124), 4, 2)])
def test_top_form_in_a_block_with_the_next_stages_first_convolution(isr, builder, shape, first, stride, layers):
    """Also where only that convolution's shifts differ, for which the block leaves its pairs."""
    builder(layers)
    test_identity_block_with_the_next_stages_first_convolution(isr, shape, first, stride)


@pytest.mark.parametrize("copies", [9, 84, 168])
def test_top_form_in_staged_rows_of_256_channels(isr, builder, copies):
    """Against the implicit-GEMM tile, in launches of few, more and many tiles."""
    builder(_TopForm)
    test_staged_rows_in_launches_of_few_and_many_tiles(isr, copies)


@pytest.mark.parametrize("in_shape,stride,copies", [((28, 28), 4, 150), ((28, 28), 1, 11), ((36, 124), 4, 13)])
def test_top_form_in_staged_rows_against_the_oracle(isr, builder, in_shape, stride, copies):
    builder(_TopForm)
    test_3x3_layers_with_staged_pixel_rows_against_the_oracle(isr, in_shape, stride, copies)


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 5, 6])
def test_top_form_in_every_conv_tile(isr, builder, tile):
    builder(_TopForm)
    test_every_conv_tile_against_the_oracle(isr, tile)


def test_top_form_in_expand_add_and_next_reduce(isr, builder):
    builder(_TopForm)
    test_expand_add_and_next_reduce_in_one_kernel(isr)


def test_clamped_layers_next_to_adds_with_and_without_halves(isr, builder):
    """The expand-and-reduce kernels in the form of layers without exact halves and nothing else, next to adds that meet some."""
    builder(_Clamped)
    test_expand_add_and_next_reduce_in_one_kernel(isr)


class _HalvesInAdds(NetBuilder):
    """Adds without rectification that meet negative exact halves: the general form of the add next to pairs of results."""

    def add(self, ta, tb, relu=True, ma=None, mb=None, sh=20, zp_out=None):
        return super().add(ta, tb, False, ma=1 << 19, mb=1 << 19, sh=20, zp_out=0 if zp_out in (None, -128) else zp_out)


class _HalvesInBoth(_HalvesInAdds):
    """The convolutions in front of them as well."""

    def conv(self, tin, cout, k, stride, pad, relu, m0=None, **kw):
        if not relu and m0 is None:
            m0 = np.full(cout, 3 << 29, dtype=np.int64)
        return super().conv(tin, cout, k, stride, pad, relu, m0=m0, **kw)


class _HalvesInBothClamped(_HalvesInBoth, _Clamped):
    """And clamps above -128: no short form anywhere."""


class _HalvesByChannel(_HalvesInAdds, _ByChannel):
    """Next to layers whose shifts differ."""


class _HalvesClamped(_HalvesInAdds, _Clamped):
    """Next to layers without exact halves and nothing else."""


@pytest.mark.parametrize("layers", [_HalvesInAdds, _HalvesInBoth, _HalvesByChannel, _HalvesClamped])
@pytest.mark.parametrize("net", ["stages", "down", "blocks of 16, 32, 64", "down-sampling blocks", "bottleneck", "bottleneck 128", "second convolution"])
def test_negative_exact_halves_that_show(isr, builder, net, layers):
    """A negative exact half is rounded away from zero, which shows only above a layer's clamp: rectified layers and sums take the forms
    without halves, so the general ones, in each kernel, run with sums that are not rectified."""
    builder(layers)
    {"stages": lambda: test_stages_of_the_nets_on_32x32_images(isr, "stages", 257),
     "down": lambda: test_stages_of_the_nets_on_32x32_images(isr, "down", 3),
     "blocks of 16, 32, 64": lambda: test_identity_residual_blocks_in_one_kernel(isr),
     "down-sampling blocks": lambda: test_downsampling_residual_blocks_in_one_kernel(isr),
     "bottleneck": lambda: test_bottleneck_blocks_in_one_kernel(isr, (30, 20)),
     "bottleneck 128": lambda: test_bottleneck_blocks_with_128_middle_channels_in_one_kernel(isr, (5, 40)),
     "second convolution": lambda: test_residual_computed_by_a_second_convolution(isr)}[net]()


@pytest.mark.parametrize("layers", [_HalvesInAdds, _HalvesByChannel, _HalvesClamped])
@pytest.mark.parametrize("copies", [11, 329])
def test_negative_exact_halves_in_expand_and_reduce(isr, builder, copies, layers):
    builder(layers)
    test_expand_and_reduce_in_launches_of_few_and_many_tiles(isr, lambda cls: None, copies, None)


@pytest.mark.parametrize("tz", [18, 20, 21, 22, 23, 26, 29, 30])
@pytest.mark.parametrize("by_channel", [False, True])
def test_exact_halves_on_both_sides_of_the_clamp(isr, tz, by_channel):
    """Multipliers (odd) * 2^tz meet exact halves (odd) / 2 steps from zero: beyond every clamp up to tz = 21, within those of zero points up to
    127, 0 and -128 + 2^(30 - tz) / 2 from 22, 23 and 30 on.  Shifts so small that the accumulators reach them."""
    _say(f"exact halves, tz {tz}, {by_channel}")
    rng = np.random.default_rng(tz)
    b = NetBuilder(rng=np.random.default_rng(91), in_shape=(3, 8, 8), num_classes=5)
    t = b.conv(b.tensor(3, 8, 8, 0, 74.0), 64, 3, 1, 1, True)
    for sh in (3, 8):
        for zp in (127, 0, -126, -128):
            odd = rng.integers(1 << (29 - tz), 1 << (30 - tz), size=64) * 2 + 1 if tz < 30 else np.ones(64, dtype=np.int64)
            shifts = np.full(64, sh) + (np.arange(64) % 3 if by_channel else 0)
            for relu in (False, True):
                u = b.conv(t, 64, 1, 1, 0, relu, m0=odd << tz, sh=shifts, zp_out=zp)
            t = b.conv(b.add(u, b.conv(t, 64, 1, 1, 0, False, m0=odd << tz, sh=shifts, zp_out=zp), True), 64, 1, 1, 0, True)
    b.fc(b.gap(t), 5)
    x = np.random.default_rng(92).integers(0, 256, size=(3, 8, 8)).astype(np.uint8)
    _check_all_tensors(isr, b.blob(), x, 64, sample=2, chunk=3)


# ---- S6-S8: logits, votes, decisions -----------------------------------------

def test_config0_full_certify_and_predict(isr):
    _say("config 0 full certify")
    blob, x = synth.build_model(0), synth.make_image(0, 1)
    om = oracle.Model(blob)
    m = _load(isr, blob, 300)
    res, c0, c1 = isr.isr_certify(m, x, 32, 100, 1000, ALPHA, seed=0, image_id=0)
    cls, rad, p_l, k, oc0, oc1 = oracle.certify(om, x, 32, 100, 1000, ALPHA, seed=0, image=0)
    assert np.array_equal(c0, oc0) and np.array_equal(c1, oc1)
    assert res.cls == cls and res.n_top == k
    assert res.p_lower == pytest.approx(p_l, rel=1e-12)
    assert res.radius == pytest.approx(rad, rel=1e-9)
    # integer-only tail (Thm 3.2, proof steps 2-3) from the device tallies, in the same call
    assert (res.cls, res.radius_int, res.radius_sq_int) == oracle.stats.certify_decision_integer(oc0, oc1, 32, 1000, ALPHA)
    assert res.radius_int > 0 and res.radius_sq_int == res.radius_int ** 2 and res.radius_int <= res.radius
    lg, am, cnt = isr.isr_debug_forward(m, x, 32, 0, 0, 1, 0, 1000)
    olg, oam, ocnt = om.mc(x, 32, 0, 0, 1, 0, 1000)
    assert np.array_equal(lg, olg) and np.array_equal(am, oam) and np.array_equal(cnt, ocnt)
    assert np.array_equal(cnt, c1)
    pres, pc = isr.isr_predict(m, x, 32, 1000, ALPHA, seed=9, image_id=2)
    pcls, pv, n_a, n_b, opc = oracle.predict(om, x, 32, 1000, ALPHA, seed=9, image=2)
    assert np.array_equal(pc, opc) and (pres.cls, pres.n_top, pres.n_second) == (pcls, n_a, n_b)
    assert pres.p_lower == pytest.approx(pv, rel=1e-9, abs=1e-300)
    m.close()


def test_votes_invariant_to_chunk_size_and_ragged_tail(isr):
    _say("chunk invariance")
    blob, x = synth.build_model(0), synth.make_image(0, 1)
    ref = None
    for chunk in (1, 7, 64, 257, 1000):
        m = _load(isr, blob, chunk)
        lg, am, cnt = isr.isr_debug_forward(m, x, 128, 4, 5, 0, 3, 333)
        cur = (lg.copy(), am.copy(), cnt.copy())
        if ref is None:
            ref = cur
            om = oracle.Model(blob)
            olg, oam, ocnt = om.mc(x, 128, 4, 5, 0, 3, 333)
            assert np.array_equal(lg, olg) and np.array_equal(am, oam) and np.array_equal(cnt, ocnt)
        else:
            assert all(np.array_equal(a, b) for a, b in zip(ref, cur))
        assert np.array_equal(np.bincount(am, minlength=m.classes).astype(np.uint32), cnt)
        m.close()


def test_fused_and_unfused_kernels_agree(isr):
    """Residual adds folded into the convolution epilogue vs one kernel per op:
    identical logits, and both equal the oracle."""
    _say("fusion on/off")
    for cfg, size, sigma in ((1, None, 64), (3, 64, 128)):
        blob = synth.build_model(cfg, size=size)
        shape = (3, size, size) if size else None
        x = synth.make_image(cfg, 2, shape=shape)
        m = _load(isr, blob, 16)
        a = isr.isr_debug_forward(m, x, sigma, 8, 2, 1, 40, 24)
        isr.isr_set_fusion(m, False)
        b = isr.isr_debug_forward(m, x, sigma, 8, 2, 1, 40, 24)
        isr.isr_set_fusion(m, True)
        assert all(np.array_equal(u, v) for u, v in zip(a, b))
        om = oracle.Model(blob)
        olg, oam, ocnt = om.mc(x, sigma, 8, 2, 1, 40, 24)
        assert np.array_equal(a[0], olg) and np.array_equal(a[1], oam) and np.array_equal(a[2], ocnt)
        m.close()


@pytest.mark.parametrize("item,sigma", [(1, 32), (1, 64), (1, 128), (2, 32), (2, 64), (2, 128)])
def test_resnet20_logits_and_votes(isr, item, sigma):
    """Two images at the three noise levels of the CIFAR-shaped workload: every selection sample
    (n0 = 100), the first 5000 and the last 300 estimation samples of an n = 100000 run --
    per-sample logits, argmax and tallies against the oracle."""
    _say(f"resnet20 logits parity image {item} sigma {sigma}")
    blob = synth.build_model(1)
    om = oracle.Model(blob)
    m = _load(isr, blob, 2048)
    x = synth.make_image(1, item)
    for phase, begin, count in ((0, 0, 100), (1, 0, 5000), (1, 99700, 300)):
        lg, am, cnt = isr.isr_debug_forward(m, x, sigma, 0, item, phase, begin, count)
        olg, oam, ocnt = om.mc(x, sigma, 0, item, phase, begin, count)
        assert np.array_equal(lg, olg) and np.array_equal(am, oam) and np.array_equal(cnt, ocnt)
    m.close()


def test_resnet20_certify_and_predict_end_to_end(isr):
    """Alg. 1 and Alg. 2 as whole calls on ResNet-20 (n0 = 100, n = 1500; chunk 700 leaves a
    ragged last chunk): tallies, selected class, bound and radius against the oracle."""
    _say("resnet20 end-to-end certify / predict")
    blob = synth.build_model(1)
    om = oracle.Model(blob)
    m = _load(isr, blob, 700)
    x = synth.make_image(1, 4)
    res, c0, c1 = isr.isr_certify(m, x, 64, 100, 1500, ALPHA, seed=11, image_id=4)
    cls, rad, p_l, k, oc0, oc1 = oracle.certify(om, x, 64, 100, 1500, ALPHA, seed=11, image=4)
    assert np.array_equal(c0, oc0) and np.array_equal(c1, oc1)
    assert res.cls == cls and res.n_top == k
    assert res.p_lower == pytest.approx(p_l, rel=1e-12)
    assert res.radius == pytest.approx(rad, rel=1e-9)
    assert (res.cls, res.radius_int, res.radius_sq_int) == oracle.stats.certify_decision_integer(oc0, oc1, 64, 1500, ALPHA)
    pres, pc = isr.isr_predict(m, x, 128, 333, ALPHA, seed=12, image_id=4)
    pcls, pv, n_a, n_b, opc = oracle.predict(om, x, 128, 333, ALPHA, seed=12, image=4)
    assert np.array_equal(pc, opc) and (pres.cls, pres.n_top, pres.n_second) == (pcls, n_a, n_b)
    assert pres.p_lower == pytest.approx(pv, rel=1e-9, abs=1e-300)
    m.close()


def test_resnet110_logits(isr):
    """1000 noisy copies of the deep narrow net inside bench.py's chunk of 4096 (the block-chain
    kernels with every workgroup full and a ragged last one): logits, argmax, tallies."""
    _say("resnet110 logits parity")
    blob = synth.build_model(2)
    om = oracle.Model(blob)
    m = _load(isr, blob, 4096)
    x = synth.make_image(2, 1)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 0, 1, 1, 500, 1000)
    olg, oam, ocnt = om.mc(x, 64, 0, 1, 1, 500, 1000)
    assert np.array_equal(lg, olg) and np.array_equal(am, oam) and np.array_equal(cnt, ocnt)
    m.close()


@pytest.mark.parametrize("sigma", [32, 64, 128, 256])
def test_resnet50_full_size_logits(isr, sigma):
    """ResNet-50 at 224x224, 101 classes: 64 sample indices per noise level in four disjoint
    ranges -- the selection loop, the start, the middle and the last indices of a
    100000-sample estimation loop -- on two images."""
    _say(f"resnet50 224 logits parity sigma {sigma}")
    blob = synth.build_model(4)
    om = oracle.Model(blob)
    m = _load(isr, blob, 16)
    for item, phase, begin, count in ((1, 0, 0, 16), (1, 1, 0, 16), (2, 1, 50000, 16), (2, 1, 99984, 16)):
        x = synth.make_image(4, item)
        lg, am, cnt = isr.isr_debug_forward(m, x, sigma, 0, item, phase, begin, count)
        olg, oam, ocnt = om.mc(x, sigma, 0, item, phase, begin, count)
        assert np.array_equal(lg, olg) and np.array_equal(am, oam) and np.array_equal(cnt, ocnt)
    m.close()


# copies of a 668-copy chunk that sit on the boundaries of the kernels' pixel tiles: first and last
# copy, both sides of the 64-, 128- and 256-copy marks (whole tiles at 7x7 ... 56x56 pixels per
# copy), the middle of the chunk (second round of workgroups), and the ragged end
CHUNK668_COPIES = (0, 1, 2, 31, 32, 63, 64, 65, 127, 128, 191, 192, 255, 256, 257, 300, 333, 334, 335, 400,
                   447, 448, 511, 512, 513, 575, 576, 639, 640, 665, 666, 667)


@pytest.mark.parametrize("sigma,item", [(32, 1), (256, 3)])
def test_resnet50_chunk_668_sampled_copies(isr, sigma, item):
    """bench.py's launch configuration (chunks of 668 copies, library-chosen tiles) at the
    smallest and the largest noise level of the headline sweep: 32 copies spread over the
    chunk, chosen on tile and workgroup-round boundaries, against the oracle one by one."""
    _say(f"resnet50 224 parity at chunk 668, sigma {sigma}")
    blob = synth.build_model(4)
    om = oracle.Model(blob)
    m = _load(isr, blob, 668)
    x = synth.make_image(4, item)
    begin = 99332                                # the last full chunk of an n = 100000 run
    lg, am, cnt = isr.isr_debug_forward(m, x, sigma, 0, item, 1, begin, 668)
    assert int(cnt.sum()) == 668 and np.array_equal(np.bincount(am, minlength=len(cnt)), cnt)
    olg, oam = _oracle_at(om, x, sigma, 0, item, 1, [begin + i for i in CHUNK668_COPIES])
    for j, i in enumerate(CHUNK668_COPIES):
        assert np.array_equal(lg[i], olg[j]) and am[i] == oam[j], i
    m.close()


def test_resnet50_in_the_benchmarked_launch_configuration(isr):
    """bench.py's configuration: chunks of 668 noisy copies, library-chosen tiles
    (256x256, 128x256, 128x128 and the fused first layer all occur).  One full chunk
    on the device; the oracle checks sampled copies one by one, the vote counts must
    add up, and forcing each tile must not change a single logit."""
    _say("resnet50 224 parity at chunk 668")
    blob = synth.build_model(4)
    om = oracle.Model(blob)
    m = _load(isr, blob, 668)
    x = synth.make_image(4, 2)
    lg, am, cnt = isr.isr_debug_forward(m, x, 128, 0, 2, 1, 20000, 668)
    assert int(cnt.sum()) == 668 and np.array_equal(np.bincount(am, minlength=len(cnt)), cnt)
    assert np.array_equal(am, np.argmax(lg, axis=1))
    picks = (0, 100, 255, 256, 333, 334, 512, 667)
    olg, oam = _oracle_at(om, x, 128, 0, 2, 1, [20000 + i for i in picks])
    for j, i in enumerate(picks):
        assert np.array_equal(lg[i], olg[j]) and am[i] == oam[j], i
    for tile in (1, 2, 3, 4, 5, 6, 7):
        _say(f"  forced tile {tile}")
        isr.isr_set_conv_tile(m, tile)
        lg2, am2, cnt2 = isr.isr_debug_forward(m, x, 128, 0, 2, 1, 20000, 668)
        assert np.array_equal(lg2, lg) and np.array_equal(cnt2, cnt)
    m.close()


@pytest.mark.parametrize("cfg,chunk", [(1, 8192), (2, 4096)])
def test_cifar_nets_in_the_benchmarked_launch_configuration(isr, cfg, chunk):
    """bench.py's configuration for the narrow nets: one full chunk (8192 / 4096 noisy
    copies) through the LDS-resident block kernels.  Votes must add up, sampled copies
    (first, last, and a few in between) are checked by the oracle one by one, and the
    op-by-op plan must give the same logits for the whole chunk."""
    _say(f"config {cfg} parity at chunk {chunk}")
    blob = synth.build_model(cfg)
    om = oracle.Model(blob)
    m = _load(isr, blob, chunk)
    x = synth.make_image(cfg, 3)
    begin = 100000 - chunk                      # the last chunk of an n = 100000 run
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 0, 3, 1, begin, chunk)
    assert int(cnt.sum()) == chunk and np.array_equal(np.bincount(am, minlength=len(cnt)), cnt)
    assert np.array_equal(am, np.argmax(lg, axis=1))
    for i in (0, 1, 4095, chunk // 2 + 1, chunk - 2, chunk - 1):
        olg, oam, _ = om.mc(x, 64, 0, 3, 1, begin + i, 1)
        assert np.array_equal(lg[i], olg[0]) and am[i] == oam[0], i
    isr.isr_set_fusion(m, False)
    lg2, am2, cnt2 = isr.isr_debug_forward(m, x, 64, 0, 3, 1, begin, chunk)
    assert np.array_equal(lg2, lg) and np.array_equal(cnt2, cnt)
    m.close()


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 5, 6, 7])
def test_every_conv_tile_against_the_oracle(isr, tile):
    """Layers deep enough for 128-byte K steps and for every output tile of the
    direct-to-LDS kernel, channel counts that leave a ragged last M tile, a ragged
    last pixel tile (37 copies of a 12x12 image), strides; tile forced through the C ABI."""
    _say(f"conv tile {tile} parity")
    rng = np.random.default_rng(51)
    b = NetBuilder(rng=np.random.default_rng(52), in_shape=(3, 12, 12), num_classes=9)
    t0 = b.tensor(3, 12, 12, 0, 74.0)
    t1 = b.conv(t0, 128, 3, 1, 1, True)
    t2 = b.conv(t1, 128, 3, 1, 1, True)                 # K = 1152
    t3 = b.conv(t2, 256, 1, 1, 0, True)                 # K = 128
    t4 = b.conv(t3, 256, 3, 1, 1, True)                 # K = 2304, 128-byte steps
    t5 = b.conv(t4, 512, 1, 1, 0, False)                # K = 256
    t6 = b.conv(t5, 272, 1, 1, 0, True)                 # K = 512, ragged M
    t7 = b.conv(t6, 320, 3, 2, 1, True)                 # K = 2448 (not a multiple of 128), stride 2, ragged M
    t8 = b.conv(t7, 1024, 1, 1, 0, True)                # K = 320
    t9 = b.conv(t8, 256, 1, 1, 0, True)                 # K = 1024, 128-byte steps, 1x1
    b.fc(b.gap(t9), 9)
    blob = b.blob()
    x = np.random.default_rng(9).integers(0, 256, size=(3, 12, 12)).astype(np.uint8)
    m = _load(isr, blob, 37)
    isr.isr_set_conv_tile(m, tile)
    om = oracle.Model(blob)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 1, 1, 1, 5, 37)
    olg, oam, ocnt = om.mc(x, 64, 1, 1, 1, 5, 37)
    assert np.array_equal(lg, olg) and np.array_equal(am, oam) and np.array_equal(cnt, ocnt)
    m.close()
    if tile == 4:
        _check_all_tensors(isr, blob, x, 64)


@pytest.mark.parametrize("copies,kernel,layers", [
    (3, "128, 128, 128, 3, 0, 1, 32x32", None), (819, "128, 128, 128, 3, 0, 1, 32x32", "_HalvesInBoth"), (819, "128, 128, 128, 3, 0, 1, 32x32", "_ByChannel"),
    (820, "128, 256, 128, 2, 0, 1, 64x32", None), (1638, "128, 256, 128, 2, 0, 1, 64x32", "_ByChannel"), (1638, "128, 256, 128, 2, 0, 1, 64x32", "_HalvesInBoth"),
    (820, "128, 256, 128, 2, 0, 1, 64x32", "_Clamped"), (4097, "128, 256, 128, 2, 0, 1, 64x64", None), (4097, "128, 256, 128, 2, 0, 1, 64x64", "_Clamped")])
def test_deep_layers_in_launches_of_few_and_many_tiles(isr, builder, copies, kernel, layers):
    """1024 -> 256 channels on 5x4 maps: sixteen waves a workgroup where all tiles run at once (at most 256 of them), the last one ragged, eight in
    launches of several rounds.  Logits that depend on every pixel: against tiles of 256 x 256, and a few copies against the oracle."""
    _say(f"deep layers, {copies} copies, {layers}")
    if layers:
        builder(globals()[layers])
    b = NetBuilder(rng=np.random.default_rng(68), in_shape=(3, 5, 4), num_classes=6)
    t = b.conv(b.conv(b.tensor(3, 5, 4, 0, 74.0), 64, 3, 1, 1, True), 1024, 1, 1, 0, True)
    b.fc(b.conv(b.conv(t, 256, 1, 1, 0, False, zp_out=-30), 16, 1, 1, 0, True), 6)
    m = _load(isr, b.blob(), copies)
    x = np.random.default_rng(69).integers(0, 256, size=(3, 5, 4)).astype(np.uint8)
    isr.isr_profile(m, 1)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 3, copies)
    names = {s["name"]: s["launches"] for s in isr.isr_profile_read(m)}
    assert names.get(f"conv_dma_kernel<{kernel}>") == 1, names
    isr.isr_set_conv_tile(m, 4)
    lg0, am0, cnt0 = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 3, copies)
    m.close()
    assert np.array_equal(lg, lg0) and np.array_equal(am, am0) and np.array_equal(cnt, cnt0)
    picks = sorted({0, 1, copies // 2, copies - 2, copies - 1})
    olg, oam = _oracle_at(oracle.Model(b.blob()), x, 64, 2, 1, 1, [3 + i for i in picks])
    assert np.array_equal(lg[picks], olg) and np.array_equal(am[picks], oam)


@pytest.mark.parametrize("in_shape,stride,copies", [((28, 28), 2, 37), ((28, 28), 4, 150), ((28, 28), 1, 11), ((12, 20), 2, 61),
                                                    ((36, 124), 4, 13), ((10, 4), 2, 333)])
def test_3x3_layers_with_staged_pixel_rows_against_the_oracle(isr, in_shape, stride, copies):
    """The 3x3 kernel that stages a tile's pixel rows once per channel slice (forced tile 7) and addresses the
    nine taps as shifted rows: its tiles of 256 consecutive pixels straddle image rows and whole images, so
    every border case of the shift arithmetic occurs -- square and non-square maps, the widest map its staging
    buffer takes (31), a map narrower than the kernel, a ragged last tile.  128-channel (64-byte slices, two
    slices) and 256-channel tiles (128-byte slices; one and two slices; a ragged second M tile).  The final
    layer is fully connected over all pixels, so one wrong activation anywhere changes the logits."""
    h, w = in_shape                                     # maps of 14x14, 7x7, 28x28, 6x10, 9x31, 5x2 behind the strided first layer
    _say(f"staged-rows 3x3 parity, input {h}x{w} stride {stride}, {copies} copies")
    b = NetBuilder(rng=np.random.default_rng(77 + h), in_shape=(3, h, w), num_classes=9)
    t0 = b.tensor(3, h, w, 0, 74.0)
    t1 = b.conv(t0, 128, 3, stride, 1, True)
    t2 = b.conv(t1, 128, 3, 1, 1, True, zp_out=-100)    # 128-channel tile, K = 1152
    t3 = b.conv(t2, 256, 3, 1, 1, False, zp_out=7)      # 256-channel tile, one slice of 128 channels
    t4 = b.conv(t3, 272, 3, 1, 1, True)                 # two slices, ragged second M tile
    t5 = b.conv(t4, 16, 1, 1, 0, True)
    b.fc(t5, 9)
    blob = b.blob()
    x = np.random.default_rng(h * 100 + w).integers(0, 256, size=(3, h, w)).astype(np.uint8)
    om = oracle.Model(blob)
    olg, oam, ocnt = om.mc(x, 64, 2, 1, 1, 3, copies)
    m = _load(isr, blob, copies)
    for tile in (7, 0):
        isr.isr_set_conv_tile(m, tile)
        lg, am, cnt = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 3, copies)
        assert np.array_equal(lg, olg) and np.array_equal(am, oam) and np.array_equal(cnt, ocnt), tile
    m.close()


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("shape,first", [((32, 56), 2), ((20, 60), 2), ((36, 124), 4)])   # 16 x 28, 10 x 30, 9 x 31
def test_identity_block_with_the_next_stages_first_convolution(isr, shape, first, stride):
    """The sum of a 256-channel block feeds the next 1x1 convolution from LDS; with a stride-2 projection as its only other
    reader (and an even height) only its even pixels are written.  Whole and ragged tiles, odd sizes."""
    _say(f"block + next 1x1 {shape} stride {stride}")
    b = NetBuilder(rng=np.random.default_rng(83), in_shape=(3,) + shape, num_classes=9)
    t = b.conv(b.conv(b.tensor(3, *shape, 0, 74.0), 64, 3, first, 1, True), 256, 1, 1, 0, True)
    u = b.conv(b.conv(b.conv(t, 64, 1, 1, 0, True), 64, 3, 1, 1, True), 256, 1, 1, 0, False)
    y = b.add(t, u, True)
    u = b.conv(b.conv(y, 128, 1, 1, 0, True), 128, 3, stride, 1, True)
    t = b.add(b.conv(y, 512, 1, stride, 0, False), b.conv(u, 512, 1, 1, 0, False), True)
    b.fc(b.conv(t, 16, 1, 1, 0, True), 9)
    blob = b.blob()
    x = np.random.default_rng(84).integers(0, 256, size=(3,) + shape).astype(np.uint8)
    m = _load(isr, blob, 5)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 3, 5)
    olg, oam, ocnt = oracle.Model(blob).mc(x, 64, 2, 1, 1, 3, 5)
    assert np.array_equal(lg, olg) and np.array_equal(am, oam) and np.array_equal(cnt, ocnt)
    m.close()
    _check_all_tensors(isr, blob, x, 64)


@pytest.mark.parametrize("copies", [1, 9, 82, 84, 165, 168])
def test_staged_rows_in_launches_of_few_and_many_tiles(isr, copies):
    """63 tiles of 256 pixels x 256 channels and fewer (64 channels a workgroup, weights three K steps ahead), 65 to 127
    (128 channels), 129 and more (256): one to four slices of 128 channels, against the implicit-GEMM tile."""
    _say(f"staged rows, {copies} copies")
    b = NetBuilder(rng=np.random.default_rng(78), in_shape=(3, 28, 28), num_classes=9)
    t = b.conv(b.tensor(3, 28, 28, 0, 74.0), 128, 3, 2, 1, True)
    t = b.conv(b.conv(b.conv(t, 256, 3, 1, 1, True), 512, 3, 1, 1, True), 256, 3, 1, 1, False)
    b.fc(b.conv(t, 16, 1, 1, 0, True), 9)
    m = _load(isr, b.blob(), copies)
    x = np.random.default_rng(79).integers(0, 256, size=(3, 28, 28)).astype(np.uint8)
    out = []
    for tile in (7, 1, 0):
        isr.isr_set_conv_tile(m, tile)
        out.append(isr.isr_debug_forward(m, x, 64, 2, 1, 1, 3, copies))
    for lg, am, cnt in out[1:]:
        assert np.array_equal(lg, out[0][0]) and np.array_equal(am, out[0][1]) and np.array_equal(cnt, out[0][2])
    m.close()


def test_expand_add_and_next_reduce_in_one_kernel(isr):
    """The kernels that run a block's closing 1x1 (128 -> 512) + residual add and the next block's opening 1x1
    (512 -> 128, or 256 for the first block of a next stage) on pixel tiles of all 512 channels.  Seven such pairs in a row (the last two with the 14x14 stage's 256 / 1024 channels): a first block whose residual is
    a stride-2 projection of the 256-channel block input issued after the closing convolution (the order of a
    ResNet-50), two identity blocks (the second with an add that meets exact halves, i.e. the other template
    instance; residual as first and as second operand), a projection block in the other order (projection
    first, stride 1), and an identity block followed by a 256-channel opening convolution.  Every tensor of one copy; then 1001 copies of a 6x6 map = 1127 tiles of 32 pixels for 512
    (256) persistent workgroups -- three and more tiles each, so the counted waits of the steady state run --
    with a ragged last tile, logits of a layer that is fully connected over all pixels, against the oracle.
    The timing report must name the kernels."""
    _say("expand + add + next reduce in one kernel")
    rng = np.random.default_rng(61)
    b = NetBuilder(rng=np.random.default_rng(62), in_shape=(3, 24, 24), num_classes=7)
    t0 = b.tensor(3, 24, 24, 0, 74.0)
    ta = b.conv(t0, 256, 3, 2, 1, True)                        # block input: 256 channels on 12x12
    u = b.conv(ta, 128, 1, 1, 0, True)
    u = b.conv(u, 128, 3, 2, 1, True)                          # 6x6
    u = b.conv(u, 512, 1, 1, 0, False, sh=rng.integers(7, 10, size=512))
    s_ = b.conv(ta, 512, 1, 2, 0, False, zp_out=-9)            # projection, stride 2, issued right before the add
    t1 = b.add(s_, u, True)
    t2 = b.conv(t1, 128, 1, 1, 0, True)                        # pair 0: projection + expand + add + t2
    t3 = b.conv(t2, 128, 3, 1, 1, True)
    t4 = b.conv(t3, 512, 1, 1, 0, False, zp_out=4, sh=rng.integers(7, 10, size=512))
    t5 = b.add(t1, t4, True)                                   # residual first
    t6 = b.conv(t5, 128, 1, 1, 0, True)                        # pair 1: t4 + add + t6
    t7 = b.conv(t6, 128, 3, 1, 1, True)
    t8 = b.conv(t7, 512, 1, 1, 0, False, sh=rng.integers(7, 10, size=512))
    t9 = b.add(t8, t5, True, ma=1 << 19, mb=1 << 19, sh=20, zp_out=-30)   # ties in the add, residual second
    t10 = b.conv(t9, 128, 1, 1, 0, True)                       # pair 2
    tb = b.conv(t10, 256, 1, 1, 0, True)                       # a block input of 256 channels on 6x6
    v = b.conv(tb, 128, 1, 1, 0, True)
    v = b.conv(v, 128, 3, 1, 1, True)
    s2 = b.conv(tb, 512, 1, 1, 0, False)                       # projection first ...
    v = b.conv(v, 512, 1, 1, 0, False, zp_out=11)              # ... the closing convolution right before the add
    t11 = b.add(v, s2, True, ma=1 << 19, mb=3 << 18, sh=20)
    t12 = b.conv(t11, 128, 1, 1, 0, True)                      # pair 3
    w_ = b.conv(t12, 128, 3, 1, 1, True)
    w_ = b.conv(w_, 512, 1, 1, 0, False)
    t13 = b.add(t11, w_, True)
    t14 = b.conv(t13, 256, 1, 1, 0, True)                      # pair 4: the next block has 256 middle channels
    # the 14 x 14 stage's shapes: 256 middle, 1024 block channels
    tc = b.conv(t14, 1024, 1, 1, 0, True)
    w_ = b.conv(tc, 256, 1, 1, 0, True)
    w_ = b.conv(w_, 256, 3, 1, 1, True)
    w_ = b.conv(w_, 1024, 1, 1, 0, False, zp_out=-3)
    t15 = b.add(tc, w_, True)
    t16 = b.conv(t15, 256, 1, 1, 0, True)                      # pair 5
    w_ = b.conv(t16, 256, 3, 1, 1, True)
    w_ = b.conv(w_, 1024, 1, 1, 0, False)
    t17 = b.add(w_, t15, True, ma=1 << 19, mb=1 << 19, sh=20)  # ties in the add
    t18 = b.conv(t17, 256, 1, 1, 0, True)                      # pair 6
    t19 = b.conv(t18, 16, 1, 1, 0, True)
    b.fc(t19, 7)
    blob = b.blob()
    x = np.random.default_rng(63).integers(0, 256, size=(3, 24, 24)).astype(np.uint8)
    _check_all_tensors(isr, blob, x, 64, sample=5, chunk=3)
    copies = 1001
    om = oracle.Model(blob)
    olg, oam, ocnt = om.mc(x, 64, 3, 2, 1, 7, copies)
    m = _load(isr, blob, copies)
    isr.isr_profile(m, 1)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 3, 2, 1, 7, copies)
    assert np.array_equal(lg, olg) and np.array_equal(am, oam) and np.array_equal(cnt, ocnt)
    stats = {s["name"]: s["launches"] for s in isr.isr_profile_read(m)}
    assert stats.get("expand_reduce_kernel<128, 512, 128>", 0) == 2, stats
    assert stats.get("proj_expand_reduce_kernel<256, 128, 512, 128>", 0) == 2, stats
    assert stats.get("expand_reduce_kernel<128, 512, 256>", 0) == 1, stats
    assert stats.get("expand_reduce_kernel<256, 1024, 256, 32 pixels>", 0) == 2, stats
    isr.isr_set_fusion(m, 0)                                   # one kernel per op gives the same
    lg0, am0, cnt0 = isr.isr_debug_forward(m, x, 64, 3, 2, 1, 7, copies)
    assert np.array_equal(lg0, olg) and np.array_equal(cnt0, ocnt)
    m.close()


@pytest.mark.parametrize("layers", [None, _ByChannel, _TopForm, _Clamped])
@pytest.mark.parametrize("copies", [1, 3, 11, 329, 656, 1000, 1967])
def test_expand_and_reduce_in_launches_of_few_and_many_tiles(isr, builder, copies, layers):
    """The four kernels on 5x5 maps, in each form of the requantisation: tiles of 32 pixels for 256 persistent workgroups, 1 to 1537 of
    them, so that a workgroup has none, one, or up to seven, the last one ragged; with 1024 channels tiles of 64 pixels where those
    take fewer rounds (329, 1000 and 1967 copies).  Logits that depend on every pixel: against one kernel per op, and three copies against the oracle."""
    _say(f"expand + reduce, {copies} copies, {layers and layers.__name__}")
    if layers:
        builder(layers)
    b = NetBuilder(rng=np.random.default_rng(64), in_shape=(3, 20, 20), num_classes=7)
    ta = b.conv(b.tensor(3, 20, 20, 0, 74.0), 256, 3, 2, 1, True)
    u = b.conv(b.conv(ta, 128, 1, 1, 0, True), 128, 3, 2, 1, True)
    u = b.conv(u, 512, 1, 1, 0, False)
    t1 = b.add(b.conv(ta, 512, 1, 2, 0, False, zp_out=-9), u, True)       # projection, stride 2
    u = b.conv(b.conv(t1, 128, 1, 1, 0, True), 128, 3, 1, 1, True)
    t2 = b.add(t1, b.conv(u, 512, 1, 1, 0, False, zp_out=4), True, ma=1 << 19, mb=1 << 19, sh=20)   # exact halves in the add
    u = b.conv(b.conv(t2, 128, 1, 1, 0, True), 128, 3, 1, 1, True)
    t3 = b.add(t2, b.conv(u, 512, 1, 1, 0, False), True)
    tc = b.conv(b.conv(t3, 256, 1, 1, 0, True), 1024, 1, 1, 0, True)
    u = b.conv(b.conv(tc, 256, 1, 1, 0, True), 256, 3, 1, 1, True)
    t4 = b.add(tc, b.conv(u, 1024, 1, 1, 0, False, zp_out=-3), True)
    u = b.conv(b.conv(t4, 256, 1, 1, 0, True), 256, 3, 1, 1, True)
    t5 = b.add(b.conv(u, 1024, 1, 1, 0, False), t4, True, ma=1 << 19, mb=1 << 19, sh=20)
    b.fc(b.conv(b.conv(t5, 256, 1, 1, 0, True), 16, 1, 1, 0, True), 7)
    m = _load(isr, b.blob(), copies)
    x = np.random.default_rng(65).integers(0, 256, size=(3, 20, 20)).astype(np.uint8)
    isr.isr_profile(m, 1)
    lg, am, cnt = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 3, copies)
    names = {s["name"]: s["launches"] for s in isr.isr_profile_read(m)}
    for kernel, launches in (("proj_expand_reduce_kernel<256, 128, 512, 128>", 1), ("expand_reduce_kernel<128, 512, 128>", 1),
                             ("expand_reduce_kernel<128, 512, 256>", 1),
                             (f"expand_reduce_kernel<256, 1024, 256, {64 if copies in (329, 1000, 1967) else 32} pixels>", 2)):
        assert names.get(kernel, 0) == launches, names
    isr.isr_set_fusion(m, 0)
    lg0, am0, cnt0 = isr.isr_debug_forward(m, x, 64, 2, 1, 1, 3, copies)
    m.close()
    assert np.array_equal(lg, lg0) and np.array_equal(am, am0) and np.array_equal(cnt, cnt0)
    few = min(3, copies)
    assert np.array_equal(lg[:few], oracle.Model(b.blob()).mc(x, 64, 2, 1, 1, 3, few)[0])


# ---- many (image, sigma) pairs in one pass -------------------------------------

def _check_batch_against_oracle(isr, m, om, xs, items, n0, n, seed):
    res, c0, c1 = isr.isr_certify_batch(m, xs, items, n0, n, ALPHA, seed=seed)
    want = oracle.certify_batch(om, xs, items, n0, n, ALPHA, seed=seed)
    for i, (cls, rad, p_l, k, oc0, oc1) in enumerate(want):
        assert np.array_equal(c0[i], oc0) and np.array_equal(c1[i], oc1), (i, items[i])
        assert res[i].cls == cls and res[i].n_top == k
        assert res[i].p_lower == pytest.approx(p_l, rel=1e-12)
        assert res[i].radius == pytest.approx(rad, rel=1e-9)
        assert (res[i].cls, res[i].radius_int, res[i].radius_sq_int) == \
            oracle.stats.certify_decision_integer(oc0, oc1, items[i][1], n, ALPHA), (i, items[i])
    pres, pc = isr.isr_predict_batch(m, xs, items, n, ALPHA, seed=seed + 1)
    pwant = oracle.predict_batch(om, xs, items, n, ALPHA, seed=seed + 1)
    for i, (cls, pv, n_a, n_b, opc) in enumerate(pwant):
        assert np.array_equal(pc[i], opc), (i, items[i])
        assert (pres[i].cls, pres[i].n_top, pres[i].n_second) == (cls, n_a, n_b)
        assert pres[i].p_lower == pytest.approx(pv, rel=1e-9, abs=1e-300)
    return res, c0, c1


@pytest.mark.parametrize("chunk", [64, 1000])
def test_batched_pairs_config0(isr, chunk):
    """Six (image, sigma) pairs over five images, four noise levels, one image used
    twice: chunks smaller than a pair's run (64) and chunks spanning several pairs
    (1000), n0 and n no multiples of either.  Every pair against the oracle, and
    against the single-pair entry point."""
    _say(f"batched certify / predict, tiny net, chunk {chunk}")
    blob = synth.build_model(0)
    om = oracle.Model(blob)
    m = _load(isr, blob, chunk)
    xs = np.stack([synth.make_image(0, i) for i in range(1, 6)])
    items = [(0, 32, 0), (1, 64, 7), (0, 128, 3), (4, 32, 9), (2, 1024, 11), (3, 64, 0)]
    res, c0, c1 = _check_batch_against_oracle(isr, m, om, xs, items, 37, 250, seed=5)
    for i, (img, sigma, image_id) in enumerate(items):
        one, s0, s1 = isr.isr_certify(m, xs[img], sigma, 37, 250, ALPHA, seed=5, image_id=image_id)
        assert np.array_equal(s0, c0[i]) and np.array_equal(s1, c1[i])
        assert (one.cls, one.n_top, one.radius, one.p_lower) == (res[i].cls, res[i].n_top, res[i].radius, res[i].p_lower)
    m.close()


def test_batched_pairs_resnet20_small_n(isr):
    """Prediction-sized runs (n = 100) of eight pairs in chunks of 512 on ResNet-20:
    five pairs share a chunk; a second call with fewer pairs reuses the buffers."""
    _say("batched certify / predict, resnet20")
    blob = synth.build_model(1)
    om = oracle.Model(blob)
    m = _load(isr, blob, 512)
    xs = np.stack([synth.make_image(1, i) for i in range(1, 5)])
    items = [(i % 4, (32, 64, 128)[i % 3], i) for i in range(8)]
    _check_batch_against_oracle(isr, m, om, xs, items, 20, 100, seed=0)
    _check_batch_against_oracle(isr, m, om, xs, items[5:7], 10, 33, seed=2)
    m.close()


@pytest.mark.parametrize("chunk", [16, 200])
def test_batched_pairs_with_the_noise_drawn_inside_the_first_layer(isr, chunk):
    """A net whose first layer is the 7x7/2 convolution + max pooling kernel, which draws the noisy
    input rows itself (no separate noise launch, the noisy copy is never stored): batched pairs over
    four images and three noise levels, chunks that split a pair's run (16) and chunks that span
    several pairs (200); every pair against the oracle and against the single-pair call; per-sample
    logits of a range against the oracle with and without the fusions."""
    _say(f"batched certify / predict, noise drawn in the first layer, chunk {chunk}")
    b = NetBuilder(rng=np.random.default_rng(33), in_shape=(3, 36, 28), num_classes=5)
    t1 = b.conv(b.tensor(3, 36, 28, 0, 74.0), 61, 7, 2, 3, True, zp_out=-100)
    t3 = b.conv(b.maxpool(t1, 3, 2, 1), 64, 1, 1, 0, True)
    b.fc(b.gap(t3), 5)
    blob = b.blob()
    om = oracle.Model(blob)
    m = _load(isr, blob, chunk)
    xs = np.stack([np.random.default_rng(40 + i).integers(0, 256, size=(3, 36, 28)).astype(np.uint8) for i in range(4)])
    items = [(0, 32, 0), (1, 64, 7), (3, 256, 3), (2, 32, 9), (0, 64, 11)]
    res, c0, c1 = _check_batch_against_oracle(isr, m, om, xs, items, 13, 57, seed=6)
    for i, (img, sigma, image_id) in enumerate(items):
        one, s0, s1 = isr.isr_certify(m, xs[img], sigma, 13, 57, ALPHA, seed=6, image_id=image_id)
        assert np.array_equal(s0, c0[i]) and np.array_equal(s1, c1[i])
    lg, am, cnt = isr.isr_debug_forward(m, xs[1], 128, 9, 4, 1, 99990, 37)
    olg, oam, ocnt = om.mc(xs[1], 128, 9, 4, 1, 99990, 37)
    assert np.array_equal(lg, olg) and np.array_equal(cnt, ocnt)
    isr.isr_set_fusion(m, False)
    lg2, _, _ = isr.isr_debug_forward(m, xs[1], 128, 9, 4, 1, 99990, 37)
    assert np.array_equal(lg2, olg)
    # the noisy copy itself is still available through the debug hook (the separate noise kernel)
    isr.isr_set_fusion(m, True)
    got = isr.isr_debug_noisy(m, xs[2], 64, 6, 9, 1, 5, 3)
    for s in range(3):
        assert np.array_equal(got[s], oracle.noisy(xs[2], 64, 6, 9, 1, 5 + s))
    m.close()


def test_tallies_of_every_size_reach_the_host(isr):
    """The last kernel's hand-over of the tallies: few, the most that the host watches for, more than that; call after call on one
    handle, so that each finds zeroed counters."""
    _say("hand-over of the tallies")
    blob = synth.build_model(0)
    m = _load(isr, blob, 256)
    om = oracle.Model(blob)
    x = synth.make_image(0, 1)
    for items in (1, 25, 26, 410, 25, 26, 1):
        pairs = [(0, 32, 7 + i) for i in range(items)]
        _, counts = isr.isr_predict_batch(m, x[None], pairs, 3, ALPHA, seed=items)
        assert counts.shape == (items, 10) and np.all(counts.sum(axis=1) == 3)
        for i in (0, items // 2, items - 1):
            assert np.array_equal(counts[i], om.mc(x, 32, items, 7 + i, 0, 0, 3)[2]), (items, i)
    m.close()


@pytest.mark.parametrize("net,chunk", [(0, 512), (0, 200), (1, 512)])
def test_votes_of_few_copies_reach_the_host_one_by_one(isr, net, chunk):
    """Calls of up to 256 copies in one chunk, whose votes the host tallies, between calls of more: predictions, both phases of a
    certification, several pairs.  Against the oracle; what one call left in the host's memory counts in no other."""
    _say(f"single votes, net {net}, chunk {chunk}")
    blob = synth.build_model(net)
    m, om = _load(isr, blob, chunk), oracle.Model(blob)
    x = synth.make_image(net, 1)
    for k, n in enumerate([256, 1, 255, 257, 201, 200, 3]):
        res, counts = isr.isr_predict(m, x, 64, n, ALPHA, seed=k, image_id=k)
        assert np.array_equal(counts, om.mc(x, 64, k, k, 0, 0, n)[2]), n
    for n0, n in [(100, 156), (100, 157), (1, 1), (20, 170)]:
        res, c0, c1 = isr.isr_certify(m, x, 32, n0, n, ALPHA, seed=n, image_id=3)
        assert np.array_equal(c0, om.mc(x, 32, n, 3, 0, 0, n0)[2]) and np.array_equal(c1, om.mc(x, 32, n, 3, 1, 0, n)[2]), (n0, n)
    for pairs, n0, n in [(5, 20, 31), (5, 20, 32), (1, 30, 40)]:
        items = [(0, 32 + i, 7 + i) for i in range(pairs)]
        _check_batch_against_oracle(isr, m, om, x[None], items, n0, n, seed=n)
    m.close()


@pytest.mark.parametrize("relu", [True, False])   # the second layer's lower clamp: -31, which has no pairs of results, and -128
@pytest.mark.parametrize("by_channel", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("classes", [2, 131])
def test_two_convolutions_as_one_kernel(isr, by_channel, classes, relu):
    """A net of two convolutions on both sides of 256 copies, where another kernel takes it, its layers' shifts equal and by channel, with
    zero points that are not zero: logits, argmax and votes against the oracle, and which kernel it was."""
    _say(f"two convolutions {by_channel} {classes} {relu}")
    b = NetBuilder(rng=np.random.default_rng(5), in_shape=(3, 32, 32), num_classes=classes)
    kw = lambda c, own: dict(sh=8 + (np.arange(c) % 3 if own else np.zeros(c, dtype=np.int64)))
    t = b.conv(b.tensor(3, 32, 32, 0, 74.0), 16, 3, 1, 1, False, zp_out=9, **kw(16, by_channel[0]))
    t = b.conv(t, 32, 3, 2, 1, relu, zp_out=-31, **kw(32, by_channel[1]))
    b.fc(b.gap(t), classes)
    blob = b.blob()
    om = oracle.Model(blob)
    m = _load(isr, blob, 320)
    x = np.random.default_rng(3).integers(0, 256, size=(3, 32, 32)).astype(np.uint8)
    for n in (257, 256, 319):
        isr.isr_profile(m, 1)
        lg, am, cnt = isr.isr_debug_forward(m, x, 64, n, 2, 1, 0, n)
        olg, oam, ocnt = om.mc(x, 64, n, 2, 1, 0, n)
        assert np.array_equal(lg, olg) and np.array_equal(am, oam) and np.array_equal(cnt, ocnt), n
        assert [k["name"] for k in isr.isr_profile_read(m)] == ["short_net_kernel" if n > 256 else "narrow_kernel<16, 32, 1, 8 waves>"], n
    m.close()


@pytest.mark.parametrize("net", [0, 1])
def test_tallies_that_the_last_workgroup_sends(isr, net):
    """Calls of more than 256 votes whose last launch is of 1 to 33 workgroups and of all (16 parts count them), with and without another
    launch before it, and of up to 256 tallies and more (10 classes, two phases, 12 pairs and 13), one behind the other: the counters
    are zero again after each, also for a call whose votes go to the host one by one.  Against the oracle."""
    _say(f"tallies of the last workgroup, net {net}")
    blob = synth.build_model(net)
    om = oracle.Model(blob)
    x = synth.make_image(net, 1)
    for chunk, ns in [(8, (257, 264, 263)), (17, (288, 289, 17, 290)), (512, (257, 272, 300, 512))]:
        m = _load(isr, blob, chunk)
        isr.isr_set_fusion(m, 2)
        for k, n in enumerate(ns):
            res, counts = isr.isr_predict(m, x, 64, n, ALPHA, seed=k, image_id=k)
            assert np.array_equal(counts, om.mc(x, 64, k, k, 0, 0, n)[2]), (chunk, n)
        m.close()
    m = _load(isr, blob, 512)
    for pairs in (12, 13, 2):
        _check_batch_against_oracle(isr, m, om, x[None], [(0, 32 + i % 5, 7 + i) for i in range(pairs)], 7, 300 // pairs, seed=pairs)
        res, c0, c1 = isr.isr_certify(m, x, 32, 20, 280, ALPHA, seed=pairs, image_id=3)
        assert np.array_equal(c0, om.mc(x, 32, pairs, 3, 0, 0, 20)[2]) and np.array_equal(c1, om.mc(x, 32, pairs, 3, 1, 0, 280)[2])
    m.close()


@pytest.mark.parametrize("chunk", [8, 1024])
def test_tallies_of_many_copies_of_a_two_convolution_net(isr, chunk):
    """Calls of more than 4096 copies, in one launch and in several, whose votes are counted in parts until the last workgroup sends them;
    batched ones of up to 256 tallies and of more in between: the counters are zero again after each.  Against the oracle."""
    _say(f"tallies of many copies, chunk {chunk}")
    blob = synth.build_model(0)
    om = oracle.Model(blob)
    x = synth.make_image(0, 1)
    m = _load(isr, blob, chunk)
    for k, n in enumerate([4097, 4096, 6001]):
        res, counts = isr.isr_predict(m, x, 64, n, ALPHA, seed=k, image_id=k)
        assert np.array_equal(counts, om.mc(x, 64, k, k, 0, 0, n)[2]), n
        res, c0, c1 = isr.isr_certify(m, x, 32, 300 + k, n, ALPHA, seed=k, image_id=3)
        assert np.array_equal(c0, om.mc(x, 32, k, 3, 0, 0, 300 + k)[2]) and np.array_equal(c1, om.mc(x, 32, k, 3, 1, 0, n)[2]), n
        pairs = (12, 13, 1)[k]
        _check_batch_against_oracle(isr, m, om, x[None], [(0, 32 + i % 5, 7 + i) for i in range(pairs)], 7, 4200 // pairs, seed=pairs)
    m.close()


@pytest.mark.parametrize("pairs,chunk,fusion", [(256, 4096, 1), (257, 4096, 1), (1, 8, 0), (2, 8, 0)])
def test_calls_in_a_row_whichever_way_they_end(isr, pairs, chunk, fusion):
    """Batched calls one right behind the other, with other noise levels and pairs each time, whose descriptors and tables go through the
    same pinned memory, on both sides of what the host watches for: 2560 tallies and more (10 classes a pair), five launches and ten
    (one chunk and two, op by op).  Against single-pair calls of a model of their own; the tallies are cleared in between."""
    _say(f"calls in a row, {pairs} pairs, chunks of {chunk}")
    blob = synth.build_model(0)
    m, other = _load(isr, blob, chunk), _load(isr, blob, 64)
    isr.isr_set_fusion(m, fusion)
    xs = np.stack([synth.make_image(0, i) for i in range(1, 4)])
    calls = [[((i + k) % 3, (16, 32, 64, 128, 256, 512)[(i + 2 * k) % 6] + k, i) for i in range(pairs)] for k in range(3)]
    import torch
    x_dev = torch.from_numpy(xs).cuda()
    got = [isr.isr_predict_batch(m, x_dev, items, 8, ALPHA, seed=k)[1] for k, items in enumerate(calls)]
    for k, items in enumerate(calls):
        assert got[k].sum() == 8 * pairs
        for i in range(0, pairs, max(1, pairs // 16)):
            want = isr.isr_predict(other, x_dev[items[i][0]], items[i][1], 8, ALPHA, seed=k, image_id=items[i][2])[1]
            assert np.array_equal(got[k][i], want), (k, i)
    m.close()
    other.close()


def test_calls_that_upload_are_refused_on_a_stream_being_captured(isr):
    """A noise level that is not resident, and a batch: nothing is recorded, and the tables are right in the calls afterwards."""
    import torch
    _say("calls under capture")
    blob = synth.build_model(0)
    om = oracle.Model(blob)
    x = synth.make_image(0, 1)
    x_dev = torch.from_numpy(x).cuda()
    m = isr.isr_load_model(blob)
    stream = torch.cuda.Stream()
    isr.isr_set_workspace(m, 64, stream=stream)
    torch.cuda.synchronize()
    isr.isr_predict_batch(m, x_dev[None], [(0, 32, 2)], 20, ALPHA, seed=1)   # its buffers are there
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        graph.capture_begin()
        unused = x_dev.clone()
        for call in (lambda: isr.isr_predict(m, x_dev, 64, 20, ALPHA, seed=1, image_id=2),
                     lambda: isr.isr_predict_batch(m, x_dev[None], [(0, 128, 2)], 20, ALPHA, seed=1)):
            with pytest.raises(isr.IsrError):
                call()
        graph.capture_end()
    torch.cuda.synchronize()
    for sigma in (64, 128, 32):
        assert np.array_equal(isr.isr_predict(m, x_dev, sigma, 20, ALPHA, seed=1, image_id=2)[1], om.mc(x, sigma, 1, 2, 0, 0, 20)[2]), sigma
        assert np.array_equal(isr.isr_predict_batch(m, x_dev[None], [(0, sigma, 2)], 20, ALPHA, seed=1)[1][0], om.mc(x, sigma, 1, 2, 0, 0, 20)[2]), sigma
    m.close()


def test_batched_call_argument_errors(isr):
    blob = synth.build_model(0)
    m = _load(isr, blob, 32)
    xs = np.stack([synth.make_image(0, i) for i in range(1, 3)])
    for items in ([(2, 32, 0)], [(0, 0, 0)], [(0, 1025, 0)], [(0, s, 0) for s in range(1, 10)]):
        with pytest.raises(isr.IsrError) as e:
            isr.isr_predict_batch(m, xs, items, 10, ALPHA)
        assert e.value.status == isr.ISR_ERR_ARG
    with pytest.raises(isr.IsrError):
        isr.isr_certify_batch(m, xs, [(0, 32, 0)], 0, 10, ALPHA)
    # eight distinct noise levels are the limit and work
    res, c = isr.isr_predict_batch(m, xs, [(1, s, 3) for s in (1, 2, 3, 4, 5, 6, 7, 8)], 40, ALPHA)
    assert all(int(row.sum()) == 40 for row in c)
    m.close()


# ---- argument handling --------------------------------------------------------

def test_error_paths(isr):
    blob, x = synth.build_model(0), synth.make_image(0, 1)
    m = isr.isr_load_model(blob)
    with pytest.raises(isr.IsrError) as e:
        isr.isr_certify(m, x, 32, 10, 10, ALPHA)
    assert e.value.status == isr.ISR_ERR_WORKSPACE
    isr.isr_set_workspace(m, 16)
    for kwargs in (dict(sigma=0), dict(sigma=1025), dict(n0=0), dict(n=0), dict(alpha=0.0), dict(alpha=1.0)):
        args = dict(sigma=32, n0=10, n=10, alpha=ALPHA)
        args.update(kwargs)
        with pytest.raises(isr.IsrError) as e:
            isr.isr_certify(m, x, args["sigma"], args["n0"], args["n"], args["alpha"])
        assert e.value.status == isr.ISR_ERR_ARG
    with pytest.raises(isr.IsrError):
        isr.isr_debug_noisy(m, x, 32, 0, 0, 0, 0, 17)   # more than the chunk
    with pytest.raises(isr.IsrError):
        isr.isr_load_model(blob[:-8])
    m.close()
