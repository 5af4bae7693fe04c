"""GPU parity of the row / elementwise kernels against the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import ops as O
from paper_2504_15465_amd import binding as B
from paper_2504_15465_amd import inputs
from gpu_util import bits_equal, bf16_close, counters, ctx, dev_bits, nan_like

pytestmark = pytest.mark.gpu


def launch(op, atom_blocks=0, count=True):
    grid, _ = B.lithos_op_grid(ctx(), op)
    total = grid[0] * grid[1] * grid[2]
    cnt = counters(total)
    if count:
        B.lithos_debug_block_counters(ctx(), cnt)
    torch.cuda.synchronize()        # torch's fills/copies run on its own stream
    try:
        B.lithos_launch_atomized(ctx(), op, (0, 0, 0), atom_blocks, None, None)
        B.lithos_partition_sync(ctx(), None)
    finally:
        B.lithos_debug_block_counters(ctx(), None)
    if count:
        assert cnt.cpu().tolist() == [1] * total
    return total


def f32_close(y, ref, tol):
    d = np.abs(y.cpu().numpy().astype(np.float64) - ref)
    assert d.max() <= tol, d.max()


@pytest.mark.parametrize("rows,cols", [(8, 4096), (128, 768), (37, 1000), (5, 2056)])
@pytest.mark.parametrize("in32,out32", [(True, True), (True, False), (False, False), (False, True)])
def test_layernorm(rows, cols, in32, out32):
    x32 = inputs.normal_f32((rows, cols), 1, 2.0, 0.5)
    g, b = inputs.normal_f32((cols,), 2, 0.02, 1.0), inputs.normal_f32((cols,), 3, 0.02)
    if in32:
        x, x64 = torch.from_numpy(x32).cuda(), x32.astype(np.float64)
    else:
        bits = inputs.to_bf16_bits(x32)
        x, x64 = dev_bits(bits), O.bf16_to_f64(bits)
    ref = O.layernorm(x64, g.astype(np.float64), b.astype(np.float64), 1e-5)
    y = nan_like((rows, cols), torch.float32 if out32 else torch.bfloat16)
    y2 = nan_like((rows, cols), torch.bfloat16) if out32 else None
    op = B.layernorm_op(x, torch.from_numpy(g).cuda(), torch.from_numpy(b).cuda(), y, rows, cols, 1e-5, y_bf16=y2)
    launch(op)
    if out32:
        f32_close(y, ref, 5e-5)
        bf16_close(y2, ref)
    else:
        bf16_close(y, ref)
    ya = nan_like(y.shape, y.dtype)
    opa = B.layernorm_op(x, torch.from_numpy(g).cuda(), torch.from_numpy(b).cuda(), ya, rows, cols, 1e-5)
    launch(opa, atom_blocks=3)
    assert bits_equal(y, ya)


@pytest.mark.parametrize("rows,cols", [(8, 4096), (16, 14336), (3, 520), (5, 1001), (70, 1024)])
@pytest.mark.parametrize("in32,out32", [(True, False), (True, True), (False, False)])
def test_rmsnorm(rows, cols, in32, out32):
    """Rows that fit in registers (cols % 4 == 0, at most 4096) take the single-read kernel,
    the others the two-pass one."""
    x32 = inputs.normal_f32((rows, cols), 4, 3.0)
    if not in32:
        x32 = O.bf16_to_f64(inputs.to_bf16_bits(x32)).astype(np.float32)
    w = inputs.normal_f32((cols,), 5, 0.1, 1.0)
    ref = O.rmsnorm(x32.astype(np.float64), w.astype(np.float64), 1e-5)
    x = torch.from_numpy(x32).cuda()
    if not in32:
        x = x.to(torch.bfloat16)
    y = nan_like((rows, cols), torch.float32 if out32 else torch.bfloat16)
    op = B.rmsnorm_op(x, torch.from_numpy(w).cuda(), y, rows, cols, 1e-5)
    launch(op)
    if out32:
        assert np.abs(y.cpu().numpy().astype(np.float64) - ref).max() <= 2e-6 * max(1.0, np.abs(ref).max())
    else:
        bf16_close(y, ref)
    ya = nan_like(y.shape, y.dtype)
    launch(B.rmsnorm_op(x, torch.from_numpy(w).cuda(), ya, rows, cols, 1e-5), atom_blocks=2)
    assert bits_equal(y, ya)


@pytest.mark.parametrize("rows,cols", [(8, 4096), (300, 3072), (7, 1001)])
@pytest.mark.parametrize("in32,out32", [(False, False), (True, True), (True, False)])
def test_bias_gelu(rows, cols, in32, out32):
    x32 = inputs.normal_f32((rows, cols), 6, 2.0)
    bias = inputs.normal_f32((cols,), 7, 0.5)
    if in32:
        x, x64 = torch.from_numpy(x32).cuda(), x32.astype(np.float64)
    else:
        bits = inputs.to_bf16_bits(x32)
        x, x64 = dev_bits(bits), O.bf16_to_f64(bits)
    ref = O.bias_act(x64, bias.astype(np.float64), gelu=True)
    y = nan_like((rows, cols), torch.float32 if out32 else torch.bfloat16)
    total = launch(B.bias_act_op(x, y, rows, cols, torch.from_numpy(bias).cuda(), gelu=True))
    assert total == (rows * cols + 2047) // 2048
    if out32:
        f32_close(y, ref, 2e-6 * max(1.0, np.abs(ref).max()))
    else:
        # fp32 erf is good to ~2e-7 absolute, so GELU's far negative tail
        # (u/2 * (1 + erf) with 1 + erf ~ 1e-6) carries ~1e-6 absolute error
        bf16_close(y, ref, abs_tol=1e-6)
    ya = nan_like(y.shape, y.dtype)
    launch(B.bias_act_op(x, ya, rows, cols, torch.from_numpy(bias).cuda(), gelu=True), atom_blocks=2)
    assert bits_equal(y, ya)


@pytest.mark.parametrize("rows,n", [(1536, 128), (9, 2049), (4, 1000)])
def test_softmax(rows, n):
    s32 = inputs.normal_f32((rows, n), 8, 3.0)
    ref = O.softmax(s32.astype(np.float64) * 0.125)
    p = nan_like((rows, n), torch.float32)
    launch(B.softmax_op(torch.from_numpy(s32).cuda(), p, rows, n, scale=0.125))
    f32_close(p, ref, 2e-6)
    assert abs(float(p.sum(dim=1).max()) - 1.0) < 1e-5
    bits = inputs.to_bf16_bits(s32)
    pb = nan_like((rows, n), torch.bfloat16)
    launch(B.softmax_op(dev_bits(bits), pb, rows, n, scale=0.125), atom_blocks=5)
    bf16_close(pb, O.softmax(O.bf16_to_f64(bits) * 0.125))


@pytest.mark.parametrize("n", [77, 1000, 1024, 2048])
def test_softmax_of_masked_and_far_apart_scores(n):
    """Rows with masked scores (-inf and the type's lowest value), with subnormal and vanishing probabilities, and
    with every score masked (NaN).  The difference to the maximum (60 +- 10) rounds to 2^-18, which is the probability's
    relative error, on top of 2e-6; or the smallest normal number where the probability is below it."""
    rng = np.random.default_rng(n)
    s = rng.normal(0.0, 2.0, (6, n)).astype(np.float32)
    s[0, ::3] = -np.inf
    s[1, 1:] = np.finfo(np.float32).min
    s[2] = np.linspace(0.0, -120.0, n)
    s[3, n // 2] = 60.0
    s[4] = -np.inf
    p = nan_like((6, n), torch.float32)
    launch(B.softmax_op(torch.from_numpy(s).cuda(), p, 6, n, scale=1.0))
    got = p.cpu().numpy().astype(np.float64)
    assert np.isnan(got[4]).all()
    rows = [0, 1, 2, 3, 5]
    ref = O.softmax(s[rows].astype(np.float64))
    assert (np.abs(got[rows] - ref) <= (2e-6 + 2.0 ** -18) * ref + np.finfo(np.float32).tiny).all()


@pytest.mark.parametrize("rows,f", [(8, 14336), (3, 1000)])
def test_silu_mul(rows, f):
    bits = inputs.normal_bits((rows, 2 * f), 9, 2.0)
    gu = O.bf16_to_f64(bits)
    ref = O.silu_mul(gu[:, :f], gu[:, f:])
    y = nan_like((rows, f), torch.bfloat16)
    launch(B.silu_mul_op(dev_bits(bits), y, rows, f), atom_blocks=4)
    bf16_close(y, ref)


@pytest.mark.parametrize("rows,n_q,n_kv,d,pos", [(4, 32, 8, 128, 2048), (3, 4, 2, 16, 5), (1, 8, 8, 64, 0)])
def test_rope_and_cache_append(rows, n_q, n_kv, d, pos):
    cap = pos + 1
    bits = inputs.normal_bits((rows, (n_q + 2 * n_kv) * d), 10)
    qkv = dev_bits(bits).clone()
    kc = torch.zeros((rows, cap, n_kv, d), dtype=torch.bfloat16, device="cuda")
    vc = torch.zeros((rows, cap, n_kv, d), dtype=torch.bfloat16, device="cuda")
    launch(B.rope_kv_op(qkv, kc, vc, rows, n_q, n_kv, d, pos, cap), atom_blocks=3)
    x = O.bf16_to_f64(bits)
    q = x[:, : n_q * d].reshape(rows, n_q, d)
    k = x[:, n_q * d:(n_q + n_kv) * d].reshape(rows, n_kv, d)
    v = x[:, (n_q + n_kv) * d:].reshape(rows, n_kv, d)
    positions = np.full((rows,), pos, dtype=np.int64)
    q_ref, k_ref = O.rope(q, positions), O.rope(k, positions)
    out = qkv.cpu().to(torch.float64).numpy()
    # fp32 angle arithmetic at position 2048 is good to ~1e-4 rad: allow 2 bf16 ulp there
    def close(g, r):
        r16 = O.round_bf16(r)
        assert np.all(np.abs(g - r16) <= np.abs(r16) * 2.0 ** -6 + 2e-3)
        assert (g == r16).mean() > 0.9
    close(out[:, : n_q * d].reshape(rows, n_q, d), q_ref)
    close(out[:, n_q * d:(n_q + n_kv) * d].reshape(rows, n_kv, d), k_ref)
    # cache slot `pos` holds exactly the rotated k and the untouched v; other slots stay zero
    assert torch.equal(kc[:, pos].reshape(rows, -1), qkv[:, n_q * d:(n_q + n_kv) * d])
    assert torch.equal(vc[:, pos].reshape(rows, -1), dev_bits(bits)[:, (n_q + n_kv) * d:])
    if pos > 0:
        assert float(kc[:, :pos].abs().max()) == 0.0 and float(vc[:, :pos].abs().max()) == 0.0


def test_row_ops_refuse_bad_arguments():
    x = torch.zeros((4, 64), dtype=torch.float32, device="cuda")
    y = torch.zeros((4, 64), dtype=torch.bfloat16, device="cuda")
    bad = [
        B.layernorm_op(x, None, None, y, 4, 64),
        B.layernorm_op(x, x, x, y, 0, 64),
        B.layernorm_op(x, x, x, y, 4, 64, y_bf16=y),      # bf16 copy without fp32 main output
        B.rmsnorm_op(x, None, y, 4, 64),
        B.rope_kv_op(y, y, y, 1, 2, 1, 15, 0, 1),         # odd head width
        B.rope_kv_op(y, y, y, 1, 2, 1, 16, 3, 3),         # pos outside the cache
        B.make_op(99, (1, 1)),
    ]
    for op in bad:
        with pytest.raises(B.LithosError) as e:
            B.lithos_launch_atomized(ctx(), op)
        assert e.value.code == B.EINVAL


@pytest.mark.parametrize("rows,cols", [(1, 1), (5, 3), (9, 8), (6, 12), (3, 63), (130, 64), (70, 65), (66, 72), (5, 127), (3, 129), (4, 1023), (5, 1024), (3, 1025), (2, 1032),
                                       (3, 4095), (2, 4096), (2, 4097), (2, 4104)])
@pytest.mark.parametrize("in32,out32", [(False, False), (True, True), (True, False)])
def test_row_kernels_at_the_edges_of_their_variants(rows, cols, in32, out32):
    """Rows of one element up to and beyond the longest register-resident row, for every access width (cols a multiple
    of 8, of 4, odd) and for outputs that are only 4-byte aligned, cut in atoms of 2 blocks."""
    x32 = inputs.normal_f32((rows, cols), [31, rows, cols], 2.0, 0.5)
    if not in32:
        x32 = O.bf16_to_f64(inputs.to_bf16_bits(x32)).astype(np.float32)
    g, b = inputs.normal_f32((cols,), 32, 0.02, 1.0), inputs.normal_f32((cols,), 33, 0.02)
    x = torch.from_numpy(x32).cuda() if in32 else torch.from_numpy(x32).cuda().to(torch.bfloat16)
    gd, bd, dt = torch.from_numpy(g).cuda(), torch.from_numpy(b).cuda(), torch.float32 if out32 else torch.bfloat16
    x64, g64, b64 = x32.astype(np.float64), g.astype(np.float64), b.astype(np.float64)
    for shift in (0, 2):                       # elements: the second output buffer is not 16-byte aligned
        ys = [nan_like((rows * cols + 8,), dt)[shift:shift + rows * cols].view(rows, cols) for _ in range(3)]
        launch(B.bias_act_op(x, ys[0], rows, cols, gd, gelu=True), atom_blocks=2)
        launch(B.layernorm_op(x, gd, bd, ys[1], rows, cols, 1e-5), atom_blocks=2)
        launch(B.softmax_op(x, ys[2], rows, cols, scale=0.7), atom_blocks=2)
        refs = [O.bias_act(x64, g64, gelu=True), O.layernorm(x64, g64, b64, 1e-5), O.softmax(x64 * 0.7)]
        # fp32 arithmetic: a few roundings of values up to max |ref| (LayerNorm: of values scaled by 1/std, which
        # rows of one or three elements make as large as 1/sqrt(eps)); bf16: one step around the rounded value
        for y, ref, tol in zip(ys, refs, (2e-6, 5e-5, 2e-6)):
            if out32:
                f32_close(y, ref, tol * max(1.0, np.abs(ref).max()))
            else:
                bf16_close(y, ref, abs_tol=tol, exact_frac=0.98 if rows * cols > 500 else 0.9)


def test_gelu_over_its_whole_range():
    """Both halves of GELU against float64, and the limits.  Error of the lower half, relative: with e = 2^-24, the
    scaled error function q = 1 - sP carries about 4e absolute (reciprocal 2e, product, last step), that is
    4e / q with 1/q <= 1 + 1.78 |u| / sqrt 2; the exponent u^2/2 carries 2.5e relative (u*u, constant, sum), so
    the exponential 2.5e u^2/2 plus 2e of its own; three more products.  Upper half: u (1 - h), at most 4e / 2
    + 3e."""
    u = np.concatenate([np.linspace(-13, 13, 20000), [-60.0, -40.0, 40.0, 60.0, 3e4, 0.0]]).astype(np.float32)
    y = nan_like((1, u.size), torch.float32)
    launch(B.bias_act_op(torch.from_numpy(u).cuda(), y, 1, u.size, None, gelu=True))
    from scipy.special import erfc
    u64, e = u.astype(np.float64), 2.0 ** -24
    ref = u64 * 0.5 * erfc(-u64 / math.sqrt(2.0))
    d = np.abs(y.cpu().numpy()[0].astype(np.float64) - ref)
    lower = e * (5 + 4 * (1 + 1.26 * np.abs(u64)) + 1.25 * u64 ** 2)
    assert np.all(d <= np.abs(ref) * np.where(u < 0, lower, 5 * e) + 1e-37), np.max(d / np.maximum(np.abs(ref), 1e-37) / e)


@pytest.mark.parametrize("n", [77, 1024, 1032, 4096])
def test_softmax_exponential_is_that_of_single_precision(n):
    """With one score of 0 and the others below -30 the denominator is 1 in fp32, so the probabilities are the kernel's
    exponentials.  Error: the hardware's 2^a, one unit in the last place (2^-23), and two roundings of an argument
    within half a unit (2^-26 each, times ln 2); subnormal results are rounded once more (2^-150)."""
    rng = np.random.default_rng(n)
    s = rng.uniform(-87.0, -30.0, (1 << 20) // n * n).astype(np.float32).reshape(-1, n)
    s[::4] -= 16.0                  # a quarter of the rows down to the last subnormal number
    s[:, n // 3] = 0.0
    p = nan_like(s.shape, torch.float32)
    launch(B.softmax_op(torch.from_numpy(s).cuda(), p, s.shape[0], n, scale=1.0))
    ref = np.exp(s.astype(np.float64))
    d = np.abs(p.cpu().numpy().astype(np.float64) - ref)
    rel = 2.0 ** -23 + 2 * 2.0 ** -26 * math.log(2.0)
    assert (d <= rel * ref + 2.0 ** -150).all(), np.max((d - 2.0 ** -150) / ref)


def test_gelu_is_that_of_single_precision_at_ordinary_arguments():
    """With e = 2^-24.  u > 0: Phi lies in [1/2, 1), so its last rounding is at most e relative, the product with u as
    much, and what is added to 1/2 (less than 0.45 of Phi) or subtracted from 1 (less than 0.12 of it) carries the rest:
    2.5 e.  -1.25 < u < 0: Phi = 1/2 - d, where d carries 1.5 e (the last rounding of P, e/4 absolute or 0.8 e relative, of
    z and of the coefficients), is subtracted with a rounding of at most e/4 absolute, and the fit is 0.2 e (1.2e-8) of
    Phi away; the product with u rounds by e."""
    rng = np.random.default_rng(5)
    u = np.concatenate([rng.uniform(1e-3, 0.5, 1 << 20), rng.uniform(0.5, 14.0, 1 << 20), -rng.uniform(1e-3, 1.25, 1 << 20)]).astype(np.float32)
    y = nan_like((1, u.size), torch.float32)
    launch(B.bias_act_op(torch.from_numpy(u).cuda(), y, 1, u.size, None, gelu=True))
    from scipy.special import ndtr
    u64, e = u.astype(np.float64), 2.0 ** -24
    phi = ndtr(u64)
    rel = np.abs(y.cpu().numpy()[0].astype(np.float64) / (u64 * phi) - 1.0)
    bound = np.where(u64 > 0, 2.5 * e, e * (1.2 + (1.5 * (0.5 - phi) + 0.25) / phi))
    assert (rel <= bound).all(), (np.max(rel[u64 > 0]) / e, np.max(rel / bound))


def median_us(op):
    """Median launch time, the best of three rounds."""
    torch.cuda.synchronize()
    return min(B.lithos_time_launch(ctx(), op, 0, None, 3, 15)[1] for _ in range(3))


@pytest.mark.parametrize("cols,most", [(127, 1.8), (1025, 4.0), (4095, 4.0)])
def test_layernorm_of_odd_rows_costs_no_more_than_its_passes(cols, most):
    """Rows that no wide access fits are read three times in single elements; the next longer rows are read once
    (measured: 1.1, 1.8 and 2.2 times as long; 2.6, 6.0 and 6.4 in the register-resident form of single elements)."""
    rows = 16384
    x = torch.randn(rows * (cols + 7), device="cuda").to(torch.bfloat16)
    y, g = torch.empty_like(x), torch.randn(cols + 7, device="cuda")
    t = [median_us(B.layernorm_op(x, g, g, y, rows, c)) for c in (cols, (cols + 7) // 8 * 8)]
    assert t[0] <= most * t[1], t


def test_softmax_of_short_rows_costs_less_than_of_longer_ones():
    """A row of 33 scores is an eighth of one of 264 (measured: 0.76 of its time; 1.06 in the register-resident form)."""
    rows = 131072
    x = torch.randn(rows * 264, device="cuda").to(torch.bfloat16)
    y = torch.empty_like(x)
    t = [median_us(B.softmax_op(x, y, rows, c)) for c in (33, 264)]
    assert t[0] <= 0.91 * t[1], t


def test_bias_of_odd_rows_stays_near_the_wide_form():
    """Single elements against 16-byte accesses of nearly the same bytes (measured: 1.3 times as long; 1.8 with every
    load waited for by itself)."""
    rows = 16384
    x, b = torch.randn(rows * 1024, device="cuda").to(torch.bfloat16), torch.randn(1024, device="cuda")
    y = torch.empty_like(x)
    t = [median_us(B.bias_act_op(x, y, rows, c, b, gelu=False)) for c in (1023, 1024)]
    assert t[0] <= 1.6 * t[1], t


@pytest.mark.parametrize("rows,cols", [(9, 8), (6, 12), (5, 63), (4, 1023), (3, 1025), (2, 1032), (3, 4095), (2, 4096), (2, 4104)])
@pytest.mark.parametrize("shift", [0, 2])
def test_paired_bf16_outputs_in_every_variant(rows, cols, shift):
    """hi + lo planes of the split and of LayerNorm's bf16 copy, for every access width and for planes that are only
    4-byte aligned: hi is the rounded value, lo the rounded rest."""
    x32 = inputs.normal_f32((rows, cols), [41, rows, cols], 2.0, 0.5)
    g, b = inputs.normal_f32((cols,), 42, 0.02, 1.0), inputs.normal_f32((cols,), 43, 0.02)
    x, gd, bd = torch.from_numpy(x32).cuda(), torch.from_numpy(g).cuda(), torch.from_numpy(b).cuda()
    n = rows * cols
    planes = lambda: nan_like((2 * n + 8,), torch.bfloat16)
    buf = planes()
    pair = buf[shift:shift + 2 * n].view(2, rows, cols)
    launch(B.split_op(x, pair, rows, cols), atom_blocks=2)
    assert torch.isnan(buf[:shift].float()).all() and torch.isnan(buf[shift + 2 * n:].float()).all()
    assert torch.equal(pair[0], x.to(torch.bfloat16))
    assert torch.equal(pair[1], (x - pair[0].float()).to(torch.bfloat16))
    buf, y = planes(), nan_like((rows, cols), torch.float32)
    pair = buf[shift:shift + 2 * n].view(2, rows, cols)
    launch(B.layernorm_op(x, gd, bd, y, rows, cols, 1e-5, y_bf16=pair, split=True), atom_blocks=2)
    assert torch.isnan(buf[:shift].float()).all() and torch.isnan(buf[shift + 2 * n:].float()).all()
    ref = O.layernorm(x32.astype(np.float64), g.astype(np.float64), b.astype(np.float64), 1e-5)
    f32_close(y, ref, 5e-5 * max(1.0, np.abs(ref).max()))
    assert torch.equal(pair[0], y.to(torch.bfloat16))
    assert torch.equal(pair[1], (y - pair[0].float()).to(torch.bfloat16))
    single = nan_like((n + 8,), torch.bfloat16)[shift:shift + n].view(rows, cols)
    launch(B.layernorm_op(x, gd, bd, y, rows, cols, 1e-5, y_bf16=single), atom_blocks=2)
    assert torch.equal(single, pair[0])
