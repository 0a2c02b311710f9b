"""GPU parity of the kernel that takes fp32 products as bf16 part products
(plan strings with a=vec_m_b3): every tile through whole, split and stream-K
schedules on ragged shapes (rows and columns that do not fill a tile, odd
stage counts, padding, strides), bit-exact on small-integer data; its error
against the fp64 oracle no larger than the fp32-MFMA kernel's; operands whose
24 significand bits are all in use; and the range check: infinities, NaNs,
overflow and values near the bottom of the exponent range come out as the
fp32-MFMA kernel (dma=1) gives them."""
import numpy as np
import pytest

import oracle
from paper_2307_04941_amd import mg3m
from tests.gpu_util import assert_parity, make, run_gpu, say, to_dev

pytestmark = pytest.mark.gpu

TILES = ["tile=128x128,waves=1x4,kt=32", "tile=128x256,waves=1x8,kt=32", "tile=64x256,waves=1x8,kt=64",
         "tile=64x128,waves=1x4,kt=64", "tile=64x128,waves=1x4,kt=32", "tile=64x64,waves=1x4,kt=32",
         "tile=64x64,waves=1x4,kt=64", "tile=32x128,waves=1x4,kt=32", "tile=64x256,waves=1x8,kt=32",
         "tile=64x64,waves=4x4,kt=32", "tile=64x64,waves=2x4,kt=32", "tile=16x16,waves=16x1,kt=32", "tile=32x32,waves=8x2,kt=32"]

# (N, C, H, W, K, R, S, stride, pad), layout, misalign.  One stage; an odd
# count; 3x3 with ragged rows and columns; stride 2 with an even window: one
# tap per stage.  Then groups of eight channels (batch vectors, any batch, one
# image, misaligned buffers), single rows (three channels; any batch; one
# channel), and NCHW.
SHAPES = [((4, 64, 3, 5, 20, 1, 1, 1, 0), "HWCN", 0), ((8, 192, 7, 5, 132, 1, 1, 1, 0), "HWCN", 0),
          ((4, 64, 13, 11, 68, 3, 3, 1, 1), "HWCN", 0), ((12, 128, 9, 10, 36, 2, 3, 2, 1), "HWCN", 0),
          ((4, 16, 9, 7, 36, 3, 3, 1, 1), "HWCN", 0), ((8, 72, 5, 6, 67, 2, 5, 1, 2), "HWCN", 0),
          ((3, 24, 8, 9, 20, 3, 3, 1, 1), "HWCN", 0), ((2, 64, 6, 5, 96, 3, 1, 3, 0), "HWCN", 0),
          ((1, 40, 11, 6, 70, 3, 3, 2, 1), "HWCN", 0), ((1, 64, 9, 9, 64, 1, 1, 1, 0), "HWCN", 0),
          ((4, 64, 7, 6, 40, 3, 3, 1, 1), "HWCN", 1), ((1, 16, 7, 6, 20, 3, 3, 1, 1), "HWCN", 1),
          ((8, 3, 10, 9, 68, 5, 3, 2, 2), "HWCN", 0), ((4, 75, 6, 5, 40, 3, 3, 1, 1), "HWCN", 0),
          ((7, 13, 6, 5, 33, 3, 2, 1, 1), "HWCN", 0), ((1, 1, 9, 8, 5, 3, 3, 1, 0), "HWCN", 0),
          ((5, 2, 12, 3, 70, 1, 3, 1, 3), "HWCN", 0),
          ((3, 64, 9, 7, 68, 3, 3, 1, 1), "NCHW", 0), ((2, 32, 5, 6, 132, 2, 3, (2, 1), (0, 2)), "NCHW", 0)]


def _plan_string(shape, layout, plan):
    N, C, H, W, K, R, S, st, pd = shape
    if isinstance(st, tuple):
        return ""
    return mg3m.conv2d_fwd_f32_plan_string(N, C, H, W, K, R, S, st, pd, layout, plan)


def _is_b3(shape, plan, layout="HWCN"):
    return "a=vec_m_b3" in mg3m.conv2d_fwd_f32_plan_string(*shape, layout, plan)


def _built(shape, layout, misalign):
    """The tiles that the shape's operand form is built for."""
    N, C = shape[:2]
    groups = {"tile=64x64,waves=2x4,kt=32", "tile=16x16,waves=16x1,kt=32", "tile=32x32,waves=8x2,kt=32"}
    four = {"tile=64x64,waves=4x4,kt=32"}
    wide = {"tile=64x256,waves=1x8,kt=32"}
    if layout == "NCHW":                               # (C of whole stages, K % 4 == 0, several taps)
        own = {"tile=128x256,waves=1x8,kt=32", "tile=64x64,waves=1x4,kt=32"} | four
        return groups | own | ({"tile=64x256,waves=1x8,kt=64"} if C % 64 == 0 else set())
    slab = N % 4 == 0 and C % 32 == 0
    if slab and misalign:
        wide = set()                                   # the workspace query, for aligned buffers, refuses it
    elif slab:
        return {t for t in TILES if t not in wide and (t[-2:] == "32" or C % 64 == 0)}
    rows = {"tile=64x128,waves=1x4,kt=32", "tile=64x64,waves=1x4,kt=32", "tile=32x128,waves=1x4,kt=32"} | wide
    return groups | rows | (set() if C % 8 == 0 else four)


@pytest.mark.parametrize("case", range(len(SHAPES)))
def test_every_b3_tile_exact(case):
    shape, layout, misalign = SHAPES[case]
    x, w, st, pd = make(shape, 3300 + case, layout, dist="int")
    acc, _ = oracle.conv2d(x, w, st, pd, layout)
    ran = set()
    for tile in TILES:
        for sched in ("split=1", "split=2", "split=5", "sk=7"):
            plan = f"{tile},{sched}" + (",via=none" if layout == "NCHW" else "")
            try:
                text = "" if misalign else _plan_string(shape, layout, plan)   # (the query plans for aligned buffers)
                assert not text or "a=vec_m_b3" in text, text
                say(f"b3 {plan} {layout} {shape}")
                y = run_gpu(x, w, st, pd, layout, plan=plan, misalign=misalign)
            except mg3m.Mg3mError as e:
                assert e.status == 7, e          # the tile is not built for this form, or sk does not apply
                continue
            ran.add(tile)
            assert np.array_equal(y, acc.astype(np.float32)), f"{shape} {plan}: not bit-exact"
    assert ran == _built(shape, layout, misalign)


@pytest.mark.parametrize("Kg", [(64, 1), (64, 3), (512, 3)])
def test_b3_error_no_larger_than_fp32_mfma(Kg):
    """Root-mean-square error against fp64 on He-normal filters and clamped
    activations; the fp32-MFMA kernel on the same data is the bound."""
    C, R = Kg
    shape = (8, C, 9, 9, 64, R, R, 1, R // 2)
    x, w, st, pd = make(shape, 3400 + C + R, "HWCN")
    x = np.maximum(x, 0)
    acc, mag = oracle.conv2d(x, w, st, pd, "HWCN")
    err = []
    for plan in ("tile=64x128,waves=1x4,kt=32", "dma=1"):
        y = run_gpu(x, w, st, pd, "HWCN", plan=plan)
        assert_parity(y, acc, mag, f"{shape} {plan}")
        err.append(float(np.sqrt(np.mean((y.astype(np.float64) - acc) ** 2) / np.mean(acc ** 2))))
    say(f"C={C} R={R}: rms error b3 {err[0]:.3g}, fp32 MFMA {err[1]:.3g}")
    assert err[0] <= err[1], err


def test_b3_keeps_every_bit():
    """A filter that picks one element: y is a shifted copy of x, bit for bit,
    whatever the 24 bits; and the same with the roles of x and w exchanged."""
    rng = np.random.Generator(np.random.PCG64(3500))
    N, C, H, W, K = 4, 64, 6, 7, 64
    bits = rng.integers(0, 2**23, (H, W, C, N), dtype=np.uint32) | (rng.integers(64, 190, (H, W, C, N), dtype=np.uint32) << 23)
    x = (bits | (rng.integers(0, 2, bits.shape, dtype=np.uint32) << 31)).view(np.float32)
    w = np.zeros((3, 3, C, K), np.float32)
    for k in range(K):
        w[k % 3, (k // 3) % 3, (5 * k) % C, k] = 1.0
    plan = "tile=64x128,waves=1x4,kt=64"
    y = run_gpu(x, w, 1, 1, "HWCN", plan=plan)
    xp = np.pad(x, ((1, 1), (1, 1), (0, 0), (0, 0)))
    for k in range(K):
        assert np.array_equal(y[:, :, k], xp[k % 3:k % 3 + H, (k // 3) % 3:(k // 3) % 3 + W, (5 * k) % C]), k
    wv = x[0, 0].reshape(1, 1, C, N)                   # 1x1 filter of arbitrary bits, one-hot pixels
    e = np.zeros((8, 8, C, 4), np.float32)
    for p in range(64):
        e[p // 8, p % 8, p, :] = 1.0
    y = run_gpu(e, np.ascontiguousarray(wv), 1, 0, "HWCN", plan="tile=64x64,waves=1x4,kt=32")
    assert np.array_equal(y[:, :, :, 0].reshape(64, N), wv[0, 0])


def test_single_products_are_rounded_once():
    """One product per output (a channel, 1x1): the fp32 product, bit for bit, as the
    fp32-MFMA kernels give it; three part products of it would be dropped."""
    for N in (16, 7, 1):
        shape = (N, 1, 20, 21, 40, 1, 1, 1, 0)
        x, w, st, pd = make(shape, 3560 + N, "HWCN")
        y = run_gpu(x, w, st, pd, "HWCN")
        assert np.array_equal(y, x[:, :, 0][:, :, None] * w[0, 0, 0][None, None, :, None]), N


def _special(kind, x, w):
    x, w = x.copy(), w.copy()
    if kind == "inf":
        x[3, 2, 5, 1] = np.inf
        x[0, 0, 0, 0] = -np.inf
    elif kind == "nan":
        x[3, 2, 5, 1] = np.nan
    elif kind == "inf_filter":
        w[1, 1, 7, 3] = np.inf
    elif kind == "near_max":                           # rounds to infinity in bf16, not in fp32
        x[3, 2, 5, 1] = np.float32(3.4e38)
        w[:] *= np.float32(1e-3)
    elif kind == "overflow":
        x *= np.float32(1e30)
        w *= np.float32(1e20)
    elif kind == "tiny":                               # parts would fall below the denormal range
        x *= np.float32(2.0**-116)
    elif kind == "tiny_sums":
        x *= np.float32(2.0**-70)
        w *= np.float32(2.0**-70)
    return x, w


@pytest.mark.parametrize("shape,plan", [((4, 16, 6, 5, 68, 3, 3, 1, 1), "tile=64x128,waves=1x4,kt=32"),
                                        ((1, 40, 6, 5, 36, 3, 3, 1, 1), "tile=64x64,waves=1x4,kt=32"),
                                        ((5, 24, 6, 5, 36, 3, 3, 1, 1), "tile=32x128,waves=1x4,kt=32"),
                                        ((4, 3, 6, 5, 68, 3, 3, 1, 1), "tile=64x64,waves=1x4,kt=32"),
                                        ((3, 5, 6, 5, 36, 3, 3, 1, 1), "tile=64x256,waves=1x8,kt=32")])
def test_b3_range_check_other_forms(shape, plan):
    """One infinity in x and in w: exactly the outputs they reach are not finite,
    the others stay within the fp32 bound (the second computation addresses its
    operands by the same forms)."""
    assert _is_b3(shape, plan)
    x, w, st, pd = make(shape, 3650, "HWCN")
    clean, mag = oracle.conv2d(x, w, st, pd, "HWCN")
    x[3, 2, shape[1] - 1, 0] = np.inf
    w[1, 2, 0, 3] = np.inf
    y = run_gpu(x, w, st, pd, "HWCN", plan=plan)
    ref = run_gpu(x, w, st, pd, "HWCN", plan="tile=64x64,waves=1x1,kt=16")
    assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isinf(y), np.isinf(ref))
    assert np.isinf(y).any() and np.isfinite(y).any()
    fin = np.isfinite(ref)
    assert np.all(np.abs(y[fin] - clean[fin]) <= 1e-5 * mag[fin])


# One plan of every operand form, of every number of groups of waves, and the
# resident-filter kernel; each layer's reduction reaches every group.
LOST_FORMS = [((4, 64, 6, 5, 68, 3, 3, 1, 1), "HWCN", "tile=64x128,waves=1x4,kt=64,split=1"),
              ((4, 64, 6, 5, 68, 3, 3, 1, 1), "HWCN", "tile=128x256,waves=1x8,kt=32,split=3"),
              ((4, 64, 6, 5, 68, 3, 3, 1, 1), "HWCN", "tile=64x64,waves=2x4,kt=32,split=1"),
              ((4, 64, 6, 5, 68, 3, 3, 1, 1), "HWCN", "tile=64x64,waves=4x4,kt=32,split=1"),
              ((4, 64, 6, 5, 68, 3, 3, 1, 1), "HWCN", "tile=32x32,waves=8x2,kt=32,split=1"),
              ((4, 64, 6, 5, 68, 3, 3, 1, 1), "HWCN", "tile=16x16,waves=16x1,kt=32,split=1"),
              ((3, 64, 6, 5, 68, 3, 3, 1, 1), "NCHW", "tile=64x64,waves=1x4,kt=32,split=1,via=none"),
              ((3, 64, 6, 5, 68, 3, 3, 1, 1), "NCHW", "tile=64x64,waves=4x4,kt=32,split=1,via=none"),
              ((4, 72, 6, 5, 36, 3, 3, 1, 1), "HWCN", "tile=64x128,waves=1x4,kt=32,split=1"),
              ((5, 72, 6, 5, 36, 3, 3, 1, 1), "HWCN", "tile=64x64,waves=2x4,kt=32,split=1"),
              ((1, 72, 6, 5, 36, 3, 3, 1, 1), "HWCN", "tile=16x16,waves=16x1,kt=32,split=1"),
              ((4, 67, 6, 5, 36, 3, 3, 1, 1), "HWCN", "tile=64x64,waves=4x4,kt=32,split=1"),
              ((5, 67, 6, 5, 36, 3, 3, 1, 1), "HWCN", "tile=32x128,waves=1x4,kt=32,split=1"),
              ((4, 128, 41, 52, 68, 1, 1, 1, 0), "HWCN", "tile=64x64,waves=1x2,kt=32")]
LOST_KINDS = ["x_low", "w_low", "x_sub", "w_sub", "x_one", "w_one", "x_parts_sub", "w_parts_sub", "w_few", "w_few_big"]


def _lost(kind, x, w, layout, rng):
    """Finite operands whose bf16 parts do not hold every bit, or barely do."""
    low, high = (w, x) if kind[0] == "w" else (x, w)
    if layout == "NCHW" and "_few" in kind:
        w = w.transpose(2, 3, 1, 0)                    # (a view: [R][S][C][K])
    if kind.endswith("_low"):                          # bits below 2^-133, worth 2^-14 of the sums
        low *= np.float32(2.0**-120)
        high *= np.float32(2.0**40)
    elif kind.endswith("parts_sub"):                   # exact in two subnormal parts
        low[...] = rng.integers(-200, 200, low.shape).astype(np.float32) * np.float32(2.0**-133)
        high *= np.float32(2.0**100)
    elif "_few" in kind:                               # decayed weights, not worth a look or worth one
        w[..., ::3, :] = rng.integers(1, 1 << 14, w[..., ::3, :].shape).astype(np.float32) * np.float32(2.0**-149)
        if kind == "w_few_big":                        # whole channels that only they meet
            few = x[:, :, ::3] if layout == "HWCN" else x[:, ::3]
            x *= np.float32(2.0**-30)
            few *= np.float32(2.0**100)
            few *= np.float32(2.0**50)
    elif kind.endswith("_sub"):                        # no part holds anything
        low *= np.float32(2.0**-136)
    else:                                              # one element; the rest of its tensor zero
        at = tuple(int(rng.integers(0, n)) for n in low.shape)
        low[...] = 0
        low[at] = np.float32((1 + 2.0**-10 + 2.0**-20) * 2.0**-122)
        high *= np.float32(2.0**60)


@pytest.mark.parametrize("form", range(len(LOST_FORMS)))
def test_b3_operands_that_lose_bits(form):
    """Operands under 2^-110 against partners of any size: each output within the
    library's 1e-5 of its magnitudes, or a step of the fp32 denormals per product,
    and sums that the parts would make zero come out."""
    shape, layout, plan = LOST_FORMS[form]
    if layout == "HWCN":
        assert _is_b3(shape, plan), plan
    rng = np.random.Generator(np.random.PCG64(3680 + form))
    Kg = shape[1] * shape[5] * shape[6]
    for kind in LOST_KINDS * 2:                        # twice: other positions of the single elements
        x, w, st, pd = make(shape, int(rng.integers(1, 1 << 30)), layout)
        _lost(kind, x, w, layout, rng)
        acc, mag = oracle.conv2d(x, w, st, pd, layout)
        say(f"b3 lost bits {kind} {layout} {shape} {plan}")
        y = run_gpu(x, w, st, pd, layout, plan=plan).astype(np.float64)
        assert np.isfinite(mag).all() and (mag > 0).any(), kind
        err, tol = np.abs(y - acc), 1e-5 * mag + Kg * 2.0**-149
        assert np.all(err <= tol), f"{kind}: worst {float((err / np.maximum(tol, 1e-300)).max()):.3g} of the tolerance"


@pytest.mark.parametrize("kind", ["inf", "nan", "inf_filter", "near_max", "overflow", "tiny", "tiny_sums"])
@pytest.mark.parametrize("plan", ["tile=64x128,waves=1x4,kt=64,split=1", "tile=128x128,waves=1x4,kt=32,sk=3",
                                  "tile=64x64,waves=1x4,kt=32,split=2"])
def test_b3_range_check(kind, plan):
    import torch
    shape = (4, 64, 6, 5, 68, 3, 3, 1, 1)
    assert _is_b3(shape, plan)
    x, w, st, pd = make(shape, 3600, "HWCN")
    x, w = _special(kind, x, w)
    y = run_gpu(x, w, st, pd, "HWCN", plan=plan)
    ref = run_gpu(x, w, st, pd, "HWCN", plan="dma=1")
    say(f"{kind} {plan}: {int((~np.isfinite(ref)).sum())} non-finite outputs, {int((ref == 0).sum())} zeros")
    # a sum that overflows does so depending on its order: infinite or NaN in both
    if kind == "overflow":
        assert np.array_equal(np.isfinite(y), np.isfinite(ref))
    else:
        assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isposinf(y), np.isposinf(ref))
        assert np.array_equal(np.isneginf(y), np.isneginf(ref))
    fin = np.isfinite(y) & np.isfinite(ref)
    with np.errstate(over="ignore", invalid="ignore"):
        xs, ws = np.where(np.isfinite(x), x, 0).astype(np.float64), np.where(np.isfinite(w), w, 0).astype(np.float64)
    mag = _magnitude(np.abs(xs), np.abs(ws))
    # two fp32 sums of 576 products: 1e-5 of the magnitudes, or the fp32 denormal step
    assert np.all(np.abs(y[fin].astype(np.float64) - ref[fin]) <= 1e-5 * mag[fin] + 600 * 2.0**-149)


def _magnitude(x, w):
    xp = np.pad(x, ((1, 1), (1, 1), (0, 0), (0, 0)))
    H, W = x.shape[:2]
    out = np.zeros((H, W, w.shape[3], x.shape[3]))
    for r in range(3):
        for s in range(3):
            out += np.einsum("hwcn,ck->hwkn", xp[r:r + H, s:s + W], w[r, s])
    return out


def test_b3_fused_in_place_with_infinity():
    """relu(conv + add) with add == y: the range check recomputes a tile before
    anything of it is stored, so add is read once."""
    import torch
    shape = (4, 64, 6, 5, 68, 3, 3, 1, 1)
    x, w, st, pd = make(shape, 3700, "HWCN")
    x[2, 2, 3, 1] = np.inf
    add = np.random.Generator(np.random.PCG64(3701)).standard_normal((6, 5, 68, 4)).astype(np.float32)
    out = []
    for plan in ("tile=64x128,waves=1x4,kt=32,split=1", "tile=64x64,waves=1x1,kt=16,split=1"):
        y = to_dev(add)
        mg3m.conv2d_fwd_f32_fused(to_dev(x), to_dev(w), y, y, 1, 4, 64, 6, 5, 68, 3, 3, 1, 1, 1, 1, "HWCN", None, 0, plan)
        torch.cuda.synchronize()
        out.append(y.cpu().numpy())
    assert np.array_equal(np.isnan(out[0]), np.isnan(out[1])) and np.array_equal(np.isinf(out[0]), np.isinf(out[1]))
    fin = np.isfinite(out[1])
    assert np.isinf(out[1]).any() and np.all(np.abs(out[0][fin] - out[1][fin]) <= 1e-4)


@pytest.mark.parametrize("form", range(len(LOST_FORMS)))
def test_b3_fused_forms_at_any_alignment(form):
    """relu(conv + add) on small integers, exact, for every form: add apart, add on
    a 4-byte boundary (loaded as wide as y is stored), and in place on a y that
    lies on one (y's alignment does not change the plan)."""
    import torch
    shape, layout, plan = LOST_FORMS[form]
    N, C, H, W, K, R, S, st, pd = shape
    x, w, _, _ = make(shape, 3720 + form, layout, dist="int")
    acc, _ = oracle.conv2d(x, w, st, pd, layout)
    add = np.random.Generator(np.random.PCG64(3740 + form)).integers(-40, 40, acc.shape).astype(np.float32)
    want = np.maximum(acc.astype(np.float32) + add, np.float32(0))
    need = mg3m.conv2d_fwd_f32_hw_workspace_bytes(N, C, H, W, K, R, S, st, st, pd, pd, layout, plan)
    ws = torch.empty((need + 3) // 4, device="cuda") if need else None
    xd, wd = to_dev(x), to_dev(w)

    def at(offset, values):
        t = torch.empty(values.size + offset, device="cuda")[offset:].view(values.shape)
        t.copy_(torch.from_numpy(values))
        return t
    for name, y, d in [("apart", at(0, add), at(0, add)), ("add off", at(0, add), at(1, add)),
                       ("y off", at(3, add), at(0, add)), ("in place", at(1, add), None)]:
        say(f"b3 fused {name} {layout} {shape} {plan}")
        mg3m.conv2d_fwd_f32_fused(xd, wd, y, y if d is None else d, 1, N, C, H, W, K, R, S, st, st, pd, pd, layout,
                                  ws, need, plan)
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), want), (name, plan)


def test_b3_network_output_at_any_alignment():
    """A network's workspace is sized once, for aligned buffers: a caller's y (or x)
    on a 4-byte boundary has to do with it."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(3760)
    N, C, HW, K = 64, 176, 28, 96
    x = torch.randn((HW, HW, C, N), generator=g, device="cuda")
    w = torch.randn((3, 3, C, K), generator=g, device="cuda") * 0.05
    net = mg3m.Net([{"op": "conv", "input": 0, "add": -1, "relu": 0, "K": K, "C": C, "R": 3, "S": 3, "stride": 1, "pad": 1,
                     "w": w}], (N, C, HW, HW), "HWCN")
    y = net.forward(x)
    off = torch.empty(y.numel() + 1, device="cuda")[1:].view(y.shape)
    net.forward(x, out=off)
    assert torch.equal(off, y)                         # the same plan
    xo = torch.empty(x.numel() + 1, device="cuda")[1:].view(x.shape)
    xo.copy_(x)
    net.forward(xo, out=off)
    # two orders of 1584 products of order one
    assert float((off - y).abs().max()) <= 1e-5 * float(x.abs().max() * w.abs().max()) * 9 * C


# The persistent 1x1 kernel: ragged rows, columns that end inside a block of 32,
# an input stride, padding, every length of the reduction, work-groups whose run
# of columns reaches into a second filter tile, and more filter tiles than
# work-groups per XCD.
RES = "tile=64x64,waves=1x2,kt=32"
RES_SHAPES = [(4, 64, 67, 65, 20, 1, 1, 1, 0), (4, 128, 33, 32, 260, 1, 1, 1, 0), (12, 192, 60, 58, 70, 1, 1, 2, 1),
              (20, 384, 23, 21, 132, 1, 1, 1, 0), (4, 64, 14, 9, 2180, 1, 1, 1, 0), (8, 320, 29, 31, 129, 1, 1, 1, 0)]


@pytest.mark.parametrize("shape", RES_SHAPES)
def test_b3_resident_exact(shape):
    info = mg3m.conv2d_fwd_f32_plan_info(*shape, "HWCN", RES)
    assert info["persistent"] == 1 and info["a_mode"] == 3 and info["grid"] == 256, info
    x, w, st, pd = make(shape, 3800 + shape[1], "HWCN", dist="int")
    acc, _ = oracle.conv2d(x, w, st, pd, "HWCN")
    say(f"b3 resident {shape}")
    assert np.array_equal(run_gpu(x, w, st, pd, "HWCN", plan=RES), acc.astype(np.float32))


def test_b3_resident_error_range_and_fused():
    """Its error no larger than the fp32-MFMA kernel's; an infinity in x, one in
    w and sums near the bottom of the range, computed again by the wave that
    meets them (the patches of its next block are in flight then); and
    relu(conv + add) in place."""
    import torch
    shape = (4, 128, 33, 32, 260, 1, 1, 1, 0)
    N, C, H, W, K = shape[:5]
    x, w, st, pd = make(shape, 3900, "HWCN")
    acc, mag = oracle.conv2d(x, w, st, pd, "HWCN")
    y, ref = (run_gpu(x, w, st, pd, "HWCN", plan=p) for p in (RES, "dma=1"))
    assert_parity(y, acc, mag, f"{shape}")
    err = [float(np.sqrt(np.mean((v.astype(np.float64) - acc) ** 2) / np.mean(acc ** 2))) for v in (y, ref)]
    assert err[0] <= err[1], err

    add = np.asarray(np.random.Generator(np.random.PCG64(3901)).standard_normal((H, W, K, N)), np.float32)
    xd, wd, yd = to_dev(x), to_dev(w), to_dev(add)
    mg3m.conv2d_fwd_f32_fused(xd, wd, yd, yd, 1, N, C, H, W, K, 1, 1, 1, 1, 0, 0, "HWCN", None, 0, RES)
    torch.cuda.synchronize()
    want = y + add                               # the plain result and one fp32 addition
    assert np.array_equal(yd.cpu().numpy(), np.where(want < 0, np.float32(0), want))

    x[3, 2, 5, 1] = np.inf
    x[7] *= np.float32(2.0**-110)
    w[0, 0, 7, 3] = -np.inf
    y, ref = (run_gpu(x, w, st, pd, "HWCN", plan=p) for p in (RES, "dma=1"))
    assert np.array_equal(np.isnan(y), np.isnan(ref))
    assert np.array_equal(np.isposinf(y), np.isposinf(ref)) and np.array_equal(np.isneginf(y), np.isneginf(ref))
    fin = np.isfinite(ref)
    xs, ws = np.where(np.isfinite(x), x, 0), np.where(np.isfinite(w), w, 0)
    _, mag = oracle.conv2d(xs, ws, st, pd, "HWCN")
    # two fp32 sums of 128 products: 1e-5 of the magnitudes, or the fp32 denormal step
    assert np.all(np.abs(y[fin].astype(np.float64) - ref[fin]) <= 1e-5 * mag[fin] + 128 * 2.0**-149)
