"""GPU parity of the stateless entry points against the oracle (through the C ABI)."""
import numpy as np
import pytest
import torch

from paper_2602_21780_amd import xsv
from paper_2602_21780_amd.inputs import to_u16
from oracle import ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def randn_bf16(shape, seed, scale=1.0, outliers=()):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(shape, generator=g) * scale
    for c in outliers:
        x[..., c] *= 8.0
    return x.to(torch.bfloat16).to(DEV)


@pytest.mark.parametrize("bits,G", [(4, 64), (4, 32), (2, 64), (2, 32)])
@pytest.mark.parametrize("H,T", [(2, 64), (3, 150), (1, 1), (16, 1374)])
def test_quantize_k_and_v_bit_exact(bits, G, H, T):
    print(f"quantize bits={bits} G={G} H={H} T={T}", flush=True)
    x = randn_bf16((H, T, 64), 17 * T + bits + G, 1.5, outliers=(3, 40))
    x16 = to_u16(x)
    for fn_gpu, fn_ref in ((xsv.quantize_k, ref.quantize_k), (xsv.quantize_v, ref.quantize_v)):
        codes, scale, zero = fn_gpu(x, bits, G)
        rc, rs, rz = fn_ref(x16, bits, G)
        assert np.array_equal(codes.cpu().numpy(), rc)
        assert np.array_equal(scale.cpu().numpy(), rs)
        assert np.array_equal(zero.cpu().numpy(), rz)


def test_quantize_degenerate_groups():
    # constant groups (s = 1 fallback), groups away from zero (zero point outside the code range),
    # exact half-way values (ties to even)
    x = torch.zeros((1, 64, 64))
    x[0, :, 0] = 3.0
    x[0, :, 1] = torch.linspace(5, 6, 64)
    x[0, :, 2] = torch.arange(64) * 0.5
    x[0, 5, :] = 7.0
    xb = x.to(torch.bfloat16).to(DEV)
    for fn_gpu, fn_ref in ((xsv.quantize_k, ref.quantize_k), (xsv.quantize_v, ref.quantize_v)):
        for bits in (2, 4):
            codes, scale, zero = fn_gpu(xb, bits, 64)
            rc, rs, rz = fn_ref(to_u16(xb), bits, 64)
            assert np.array_equal(codes.cpu().numpy(), rc)
            assert np.array_equal(scale.cpu().numpy(), rs) and np.array_equal(zero.cpu().numpy(), rz)


@pytest.mark.parametrize("bits", [2, 4])
def test_quantize_quotients_on_and_next_to_rounding_boundaries(bits):
    """Groups whose scale is exactly 1, 1/2 or 3 (quotients that are exact half-integers: ties to even, and
    thirds next to them), groups far from zero (large zero points, large quotients) and tiny magnitudes: every
    code must be the one IEEE division and round-half-to-even give."""
    top = (1 << bits) - 1
    g = torch.Generator().manual_seed(5)
    x = torch.zeros((2, 256, 64))
    k = torch.randint(0, 2 * top + 1, (2, 256, 64), generator=g).float() * 0.5       # multiples of 1/2 in [0, top]
    x[:] = k
    x[:, :, 0] = 0.0
    x[:, :, 1] = float(top)                                                          # every token group spans [0, top]: s = 1
    x[0, :, 8:16] = k[0, :, 8:16] * 0.5                                              # quarters
    x[0, :, 16:24] = k[0, :, 16:24] * 3.0 + 300.0                                    # s = 3 on [300, 300 + 3 top]: zero point -100
    x[1, :, 24:32] = k[1, :, 24:32] * 2.0 ** -100                                    # tiny scale
    x[1, :, 32:40] = -4096.0 + k[1, :, 32:40]                                        # quotients in the thousands
    x[0, 0::64, :] = 0.0
    x[0, 1::64, :] = float(top)                                                      # every channel group spans at least [0, top]
    xb = x.to(torch.bfloat16).to(DEV)
    for fn_gpu, fn_ref in ((xsv.quantize_k, ref.quantize_k), (xsv.quantize_v, ref.quantize_v)):
        for G in (32, 64):
            codes, scale, zero = fn_gpu(xb, bits, G)
            rc, rs, rz = fn_ref(to_u16(xb), bits, G)
            assert np.array_equal(scale.cpu().numpy(), rs) and np.array_equal(zero.cpu().numpy(), rz)
            assert np.array_equal(codes.cpu().numpy(), rc)


@pytest.mark.parametrize("bits", [2, 4])
def test_quantize_extreme_magnitudes_next_to_ordinary_groups(bits):
    """Groups of huge (1e30), tiny (1e-30) and ordinary values side by side, per channel and per token: the
    quantizer's quotient takes its division-free form only where no intermediate can leave the normal range,
    and both forms must give the oracle's codes."""
    g = torch.Generator().manual_seed(9)
    x = torch.randn((2, 192, 64), generator=g)
    x[0, :, 5] *= 1e30
    x[0, :, 6] *= 1e-30
    x[1, 10:20, :] *= 3e25
    x[1, 100:110, :] *= 1e-28
    x[1, 64:128, 40] = 2.5e20 + x[1, 64:128, 40] * 1e18
    xb = x.to(torch.bfloat16).to(DEV)
    for fn_gpu, fn_ref in ((xsv.quantize_k, ref.quantize_k), (xsv.quantize_v, ref.quantize_v)):
        for G in (32, 64):
            codes, scale, zero = fn_gpu(xb, bits, G)
            rc, rs, rz = fn_ref(to_u16(xb), bits, G)
            assert np.array_equal(scale.cpu().numpy(), rs) and np.array_equal(zero.cpu().numpy(), rz)
            assert np.array_equal(codes.cpu().numpy(), rc)


@pytest.mark.parametrize("bits,G,T", [(4, 64, 130), (4, 32, 95), (2, 64, 64), (2, 32, 33)])
def test_cache_of_one_frame_equals_the_stateless_quantizers(bits, G, T):
    """The re-quantization of a context's cache and the stateless quantizers are two kernels: same codes, scales and zero
    points, over ordinary groups, groups that need the division (extreme magnitudes) and constant ones, ragged last groups
    - and into a codes buffer of odd address, which takes no wide stores."""
    H = 3
    x = randn_bf16((H, T, 64), 5 * T + bits, 1.5, outliers=(3, 40)).float()
    x[0, :, 7] *= 1e30
    x[1, 3, :] *= 1e-30
    x[2, :, 9] = -2.5
    x[2, 5, :] = 0.0
    x = x.to(torch.bfloat16)
    ctx = xsv.Context(1, H, 64, T, 0, 4 * T, bits, G)
    ctx.step(0, x, x, x)
    dump = ctx.cache_export(0)
    ctx.destroy()
    for name, fn, got in (("xsv_quantize_k", xsv.quantize_k, (dump.k_codes, dump.k_scale, dump.k_zero)),
                          ("xsv_quantize_v", xsv.quantize_v, (dump.v_codes, dump.v_scale, dump.v_zero))):
        codes, scale, zero = fn(x, bits, G)
        for a, b in zip((codes, scale, zero), got):
            assert np.array_equal(a.cpu().numpy(), b)
        odd = torch.zeros(codes.numel() + 3, dtype=torch.uint8, device=DEV)
        rc = getattr(xsv.lib(), name)(None, x.data_ptr(), H, T, 64, bits, G, odd.data_ptr() + 1, scale.data_ptr(), zero.data_ptr())
        assert rc == xsv.XSV_OK
        assert torch.equal(odd[1:1 + codes.numel()], codes.reshape(-1)) and odd[0] == 0 and not odd[1 + codes.numel():].any()


@pytest.mark.parametrize("bits,G", [(4, 64), (4, 32), (2, 64), (2, 32)])
def test_zeros_of_both_signs_give_the_same_zero_point_everywhere(bits, G):
    """A group whose smallest element is a zero: its zero point is +0 if a -0 is among the elements and -0 otherwise, wherever
    in the group that is - the minimum of zeros of both signs is -0 in whatever order a kernel takes it - in the cache and
    from the stateless quantizers, bit for bit."""
    H, T = 2, 256
    g = torch.Generator().manual_seed(bits + G)
    x = torch.zeros((H, T, 64))
    x[torch.rand((H, T, 64), generator=g) < 0.02] = -0.0
    x[1] = x[1] + torch.rand((T, 64), generator=g) * (torch.rand((T, 64), generator=g) < 0.5)
    x = x.to(torch.bfloat16)
    neg = torch.signbit(x.float())
    assert float(x.float().min()) == 0.0 and bool(neg.any())
    ctx = xsv.Context(1, H, 64, T, 0, 4 * T, bits, G)
    xd = x.to(DEV)
    ctx.step(0, xd, xd, xd)
    d = ctx.cache_export(0)
    ctx.destroy()
    zero = x.float() == 0
    for fn, cached, groups in ((xsv.quantize_k, d.k_zero, lambda t: t.reshape(H, T // G, G, 64).any(2)),
                               (xsv.quantize_v, d.v_zero, lambda t: t.reshape(H, T, 64 // G, G).any(3))):
        holds_zero, holds_neg = groups(zero), groups(neg)
        assert bool((holds_zero & holds_neg).any()) and bool((holds_zero & ~holds_neg).any())
        want = torch.where(holds_neg, 0.0, -0.0).view(torch.int32)
        for got in (torch.from_numpy(cached).reshape(holds_zero.shape), fn(xd, bits, G)[2].cpu()):
            assert torch.equal(got.view(torch.int32)[holds_zero], want[holds_zero])


@pytest.mark.parametrize("H,n,n_s,P,g", [(2, 64, 5, 192, 16), (16, 1374, 5, 2722, 16), (3, 37, 5, 70, 4), (1, 21, 0, 1, 1),
                                         (20, 150, 5, 333, 16), (37, 90, 3, 100, 7)])
def test_score_matches_oracle(H, n, n_s, P, g):
    print(f"score H={H} n={n} P={P}", flush=True)
    q = randn_bf16((H, n, 64), n + P)
    k = randn_bf16((H, P, 64), n + P + 1, outliers=(7, 21, 33))
    s = xsv.score(q, k, n_s, g).cpu().numpy()
    expect, _ = ref.score(to_u16(q), to_u16(k), n_s, g)
    # fp32 sums in a different order: a few ulp of the largest score
    err = float(np.max(np.abs(s - expect)))
    assert err <= 1e-6 * (1.0 + float(np.abs(expect).max())), err
    # strided query tensor (a view into a larger buffer) gives the same bits
    big = torch.zeros((H, n, 128), dtype=torch.bfloat16, device=DEV)
    big[:, :, :64] = q
    s2 = xsv.score(big[:, :, :64], k, n_s, g).cpu().numpy()
    assert np.array_equal(s, s2)


@pytest.mark.parametrize("offset", [1, 2, 3, 4, 7, 8])
@pytest.mark.parametrize("H,n,P", [(3, 37, 70), (16, 64, 333)])
def test_score_of_keys_that_begin_at_any_element(H, n, P, offset):
    """Contiguous keys anywhere in a buffer (2 to 16 bytes past a 16-byte boundary): the bits of the same keys on one."""
    print(f"score H={H} n={n} P={P} offset={offset}", flush=True)
    q = randn_bf16((H, n, 64), n + P)
    k = randn_bf16((H, P, 64), n + P + 1, outliers=(7, 21, 33))
    moved = torch.zeros(offset + H * P * 64, dtype=torch.bfloat16, device=DEV)[offset:].view(H, P, 64)
    moved.copy_(k)
    assert k.data_ptr() % 16 == 0 and moved.data_ptr() % 16 == 2 * offset % 16
    want = xsv.score(q, k, 5, 16)
    assert torch.equal(xsv.score(q, moved, 5, 16), want)
    out = torch.full_like(want, float("nan"))
    xsv.score_noalloc(q, moved, 5, 16, out)
    assert torch.equal(out, want)


@pytest.mark.parametrize("P,k", [(1, 1), (50, 0), (50, 50), (257, 100), (2722, 1348), (7151, 6110), (40000, 12345)])
def test_topk_keep_bit_exact_with_ties(P, k):
    print(f"topk P={P} k={k}", flush=True)
    g = torch.Generator().manual_seed(P)
    tied = (torch.randint(0, 50, (P,), generator=g).float() / 8 - 3).to(DEV)        # many exact ties, both signs
    smooth = torch.randn(P, generator=g).to(DEV)
    for scores in (tied, smooth):
        keep = xsv.topk_keep(scores, k, 7, 5).cpu().numpy()
        assert np.array_equal(keep, ref.select(scores.cpu().numpy(), k, 7, 5))


@pytest.mark.parametrize("P", [2, 63, 64, 65, 511, 513, 4095, 4096, 4097, 8191, 8192, 8193, 16385])
def test_topk_keep_at_the_edges_of_chunks_and_segments(P):
    """Lists around a wave's chunk of 64 scores and the 4096 / 8192 scores a workgroup holds in registers; scores that differ
    only in one of the three digits of their order keys, ties of both zeros, infinities."""
    g = torch.Generator().manual_seed(P)
    bits = torch.randint(0, 1 << 10, (P,), generator=g, dtype=torch.int32)
    low = (0x3F800000 + bits).view(torch.float32)                                   # last digit only
    middle = (0x3F800000 + (bits << 10)).view(torch.float32)                        # middle digit only
    wild = torch.randn(P, generator=g) * torch.exp2(torch.randint(-100, 100, (P,), generator=g).float())
    few = torch.tensor([0.0, -0.0, 1.0, -1.0, float("inf"), float("-inf")])[torch.randint(0, 6, (P,), generator=g)]
    for scores in (low, -middle, wild, few):
        for k in sorted({1, P // 2, P - 1}):
            keep = xsv.topk_keep(scores.to(DEV), k, 3, 2).cpu().numpy()
            key = scores.view(torch.int32).numpy().astype(np.int64)
            key = np.where(key < 0, -(key & 0x7FFFFFFF) - 1, key)                   # the order of the scores, -0 below +0
            order = np.sort(np.lexsort((np.arange(P), -key))[:k])
            assert keep.tolist() == [0, 1, 2] + (order + 3).tolist() + [P + 3, P + 4], (P, k)


def test_topk_keep_all_equal_scores_take_smallest_positions():
    scores = torch.zeros(1000, device=DEV)
    keep = xsv.topk_keep(scores, 10, 0, 0).cpu().numpy()
    assert keep.tolist() == list(range(10))


@pytest.mark.parametrize("H,n,splits", [(2, 64, 0), (3, 150, 2), (16, 1374, 0), (16, 1041, 0), (1, 1, 0)])
def test_frame_attention_matches_oracle(H, n, splits):
    """Attention inside one frame (no cache): the oracle's attention over the frame's own keys; the context's
    streaming state is not touched."""
    print(f"frame attention H={H} n={n}", flush=True)
    q, k, v = (randn_bf16((H, n, 64), 3 * n + i, outliers=((5, 50) if i == 1 else ())) for i in range(3))
    ctx = xsv.Context(1, H, 64, n, min(5, n), 4 * n, 4, 64)
    ctx.set_attend_splits(splits, splits)
    ctx.step(0, q, k, v)                         # a cached frame that frame attention must ignore
    out = ctx.frame_attend(q, k, v)
    rows = np.unique(np.array([0, n // 3, n // 2, n - 1], np.int32))
    expect = ref.attend(to_u16(q), to_u16(k), to_u16(v), 0.125, rows=rows)
    got = to_u16(out)[:, rows].astype(np.uint32) << 16
    got = got.view(np.float32).astype(np.float64)
    assert float(np.max(np.abs(got - expect))) <= 2e-2
    rms = float(np.sqrt(np.mean((got - expect) ** 2)) / np.sqrt(np.mean(expect ** 2)))
    assert rms <= 1e-2
    assert ctx.cache_len(0) == n
    ctx.step(0, q, k, v)                         # the stream goes on as if nothing had happened
    assert ctx.cache_len(0) == 2 * n
    ctx.destroy()


def cached_rows(ctx):
    """Keys and values of layer 0's cache as attention sees them (the dequantized view), in double."""
    d = ctx.cache_export(0)
    return (torch.from_numpy(x.astype(np.int32) << 16).view(torch.float32).double() for x in (d.k_bf16, d.v_bf16))


@pytest.mark.parametrize("variant,splits", [(0, 1), (1, 2), (2, 1), (3, 2)])
def test_frame_attention_of_nan_and_infinite_inputs(variant, splits):
    """A NaN key (in a full and in a ragged tile) shows in every row of its head, a query with a NaN or an infinity in its own
    row alone; a logit of +inf (in the first, a later and the ragged tile) makes its row NaN, one of -inf takes its key out of
    the row - also where a range begins with such keys only."""
    n, H = 64 * 4 + 17, 7
    g = torch.Generator().manual_seed(variant)
    q, k, v = (torch.randn((H, n, 64), generator=g) for _ in range(3))
    q[:, :, 0] = 1.0
    q[3:, 16:32, 0] = q[3:, 48:67, 0] = -1.0
    q[4, :, 0] = -1.0
    k[0, 100, 3] = float("nan")
    k[1, n - 2, 3] = float("nan")
    q[2, 5, 7] = float("nan")
    q[2, 200, 60] = float("-inf")
    k[3, 150, 0] = float("inf")
    k[5, 3, 0] = float("inf")
    k[6, n - 5, 0] = float("inf")
    k[4, :40, 0] = float("inf")
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    ctx = xsv.Context(1, H, 64, n, 5, 4 * n, 4, 64)
    ctx.set_attend_variant(variant)
    ctx.set_attend_splits(splits, splits)
    out = ctx.frame_attend(q.to(DEV), k.to(DEV), v.to(DEV)).cpu().double()
    ctx.destroy()
    qd, kd, vd = q.double(), k.double(), v.double()
    want = torch.matmul(torch.softmax(torch.matmul(qd, kd.transpose(1, 2).contiguous()) / 8.0, -1), vd)
    assert torch.equal(out.isnan(), want.isnan())
    assert [int(w.isnan().any(-1).sum()) for w in want] == [n, n, 2, n - 35, 0, n - 35, n - 35]
    err = (out - want)[~want.isnan()]
    # bf16 probabilities and outputs: each 2^-9 relative, so a value of magnitude <= 4.5 is off by at most 2 * 2^-9 * 4.5
    assert err.abs().max() <= 2e-2


@pytest.mark.parametrize("variant,splits", [(0, 1), (1, 0), (2, 3), (3, 1), (3, 0)])
@pytest.mark.parametrize("bits", [16, 4, 2])
def test_nan_products_stay_in_their_rows(bits, variant, splits):
    """Keys that are infinite in one channel, where some queries are 0, or in two, where some queries differ in sign: NaN
    logits in those rows, -inf (or NaN, for a NaN key) in the others.  The first kind leaves every other row of the head as
    if that key were absent - the rows 16 away included.  In a full and in the ragged tile of the frame, behind a cache whose
    tiles the rows attend to as well."""
    n, H = 64 * 2 + 17, 5
    g = torch.Generator().manual_seed(7 * variant + bits)
    q, k, v, k0, v0 = (torch.randn((H, n, 64), generator=g) for _ in range(5))
    inf = float("inf")
    q[:, :, :2] = -1.0
    q[0, 5, 0] = q[0, 77, 0] = 0.0
    k[0, 20, 0] = inf
    q[1, 40, 1] = 1.0
    k[1, 70, :2] = inf
    q[2, 127, 0] = 0.0
    k[2, n - 2, 0] = inf
    k[3, 9, 30] = float("nan")
    q[4, n - 1, 0] = 0.0
    k[4, [3, 66, n - 1], 0] = inf
    q, k, v, k0, v0 = (x.to(torch.bfloat16) for x in (q, k, v, k0, v0))
    ctx = xsv.Context(1, H, 64, n, 0, 4 * n, bits, 64)
    ctx.set_attend_variant(variant)
    ctx.set_attend_splits(splits, splits)
    ctx.step(0, q.to(DEV), k0.to(DEV), v0.to(DEV))
    kc, vc = cached_rows(ctx)
    out = ctx.step(0, q.to(DEV), k.to(DEV), v.to(DEV)).cpu().double()
    ctx.destroy()
    kd, vd = torch.cat([kc, k.double()], 1), torch.cat([vc, v.double()], 1)
    want = torch.matmul(torch.softmax(torch.matmul(q.double(), kd.transpose(1, 2).contiguous()) / 8.0, -1), vd)
    assert [w.isnan().any(-1).nonzero().flatten().tolist() for w in want] == [[5, 77], [40], [127], list(range(n)), [n - 1]]
    assert torch.equal(out.isnan(), want.isnan())
    # bf16 probabilities and outputs: each 2^-9 relative, so a value of magnitude <= 4.5 is off by at most 2 * 2^-9 * 4.5
    assert (out - want)[~want.isnan()].abs().max() <= 2e-2


@pytest.mark.parametrize("variant", [0, 1, 2, 3])
@pytest.mark.parametrize("jump", [30.0, 59.0, 61.0, 140.0])
def test_frame_attention_when_the_softmax_reference_has_to_move(variant, jump):
    """A key `jump` powers of two above all keys before it, for every other query row (the rest of the wave's rows keep
    their reference): inside the first tile, in a later one, twice in a row, and in a ragged last tile - below and above
    the 60 powers of two of headroom the kernel starts a range with."""
    n, H = 64 * 4 + 17, 3
    g = torch.Generator().manual_seed(int(jump))
    q = torch.zeros((H, n, 64))
    q[:, ::2, 0] = 8.0
    q[:, :, 1:] = 0.25 * torch.randn((H, n, 63), generator=g)
    k = 0.5 * torch.randn((H, n, 64), generator=g)
    step = jump / (8.0 * 0.125 * 1.4426950408889634)            # q.k / 8 * log2(e) of channel 0 = jump
    k[:, :, 0] = 0.0
    for h, places in enumerate(([40], [70, 199], [130, n - 3])):
        for i, t in enumerate(places):
            k[h, t, 0] = step * (i + 1)
    v = torch.randn((H, n, 64), generator=g)
    q, k, v = (x.to(torch.bfloat16).to(DEV) for x in (q, k, v))
    ctx = xsv.Context(1, H, 64, n, 5, 4 * n, 4, 64)
    ctx.set_attend_variant(variant)
    ctx.set_attend_splits(1, 1)
    out = ctx.frame_attend(q, k, v).double()
    ctx.destroy()
    qd, kd, vd = q.double(), k.double(), v.double()
    want = torch.matmul(torch.softmax(torch.matmul(qd, kd.transpose(1, 2).contiguous()) / 8.0, -1), vd)
    err = out - want
    # bf16 probabilities and outputs: each 2^-9 relative, so a value of magnitude <= 4.5 is off by at most 2 * 2^-9 * 4.5
    assert err.abs().max() <= 2e-2 and err.norm() <= 1e-2 * want.norm()


@pytest.mark.parametrize("variant", [0, 1, 2, 3])
@pytest.mark.parametrize("jump", [40.0, 62.0, 100.0])
def test_infinite_values_where_the_softmax_reference_moves(variant, jump):
    """A key `jump` powers of two above all keys before it, for every other query row, with an infinite value before it, beside
    it in its tile and behind it: infinite (of that sign) in every row's channel, NaN where a channel has infinities of both
    signs or a NaN, and the other channels as they are - in the rows whose reference moves and in their neighbours."""
    n, H = 64 * 3 + 17, 5
    g = torch.Generator().manual_seed(int(jump))
    q = torch.zeros((H, n, 64))
    q[:, ::2, 0] = 8.0
    q[:, :, 1:] = 0.25 * torch.randn((H, n, 63), generator=g)
    k = 0.5 * torch.randn((H, n, 64), generator=g)
    k[:, :, 0] = 0.0
    k[:, 100, 0] = jump / (8.0 * 0.125 * 1.4426950408889634)   # q.k / 8 * log2(e) of channel 0 = jump
    v = torch.randn((H, n, 64), generator=g)
    inf = float("inf")
    v[0, 90, 7] = inf
    v[1, 3, 20] = v[1, 110, 20] = -inf
    v[2, 70, 33], v[2, 120, 33] = inf, -inf
    v[3, 180, 0] = inf
    v[4, 100, 63], v[4, 5, 2] = float("nan"), inf
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    ctx = xsv.Context(1, H, 64, n, 5, 4 * n, 4, 64)
    ctx.set_attend_variant(variant)
    ctx.set_attend_splits(1, 1)
    out = ctx.frame_attend(q.to(DEV), k.to(DEV), v.to(DEV)).cpu().double()
    ctx.destroy()
    want = torch.matmul(torch.softmax(torch.matmul(q.double(), k.double().transpose(1, 2).contiguous()) / 8.0, -1), v.double())
    assert int(want.isinf().sum()) == 4 * n and int(want.isnan().sum()) == 2 * n
    assert torch.equal(out.isnan(), want.isnan()) and torch.equal(out.isinf(), want.isinf())
    assert torch.equal(out[want.isinf()], want[want.isinf()])
    # bf16 probabilities and outputs: each 2^-9 relative, so a value of magnitude <= 4.5 is off by at most 2 * 2^-9 * 4.5
    assert (out - want)[want.isfinite()].abs().max() <= 2e-2


def frame_attention(q, k, v, variant, splits):
    H, n, _ = q.shape
    ctx = xsv.Context(1, H, 64, n, 0, 4 * n, 4, 64)
    ctx.set_attend_variant(variant)
    ctx.set_attend_splits(splits, splits)
    out = ctx.frame_attend(q.to(DEV), k.to(DEV), v.to(DEV)).cpu().double()
    ctx.destroy()
    want = torch.matmul(torch.softmax(torch.matmul(q.double(), k.double().transpose(1, 2).contiguous()) / 8.0, -1), v.double())
    return out, want


@pytest.mark.parametrize("variant,splits", [(0, 1), (1, 2), (2, 1), (3, 2)])
@pytest.mark.parametrize("power", [-120, -110, -95, -70, 60, 100])
def test_values_of_every_magnitude(variant, splits, power):
    """Values of one head, or of one channel, times 2^power: the same result times 2^power."""
    n, H = 64 * 8 + 17, 2
    g = torch.Generator().manual_seed(variant)
    q, k, v = (torch.randn((H, n, 64), generator=g) for _ in range(3))
    v[0] *= 2.0 ** power
    # one channel: only where every element is normalized by itself - a row of a cut unit's partial has a common exponent
    if splits == 1:
        v[1, :, 5] *= 2.0 ** power
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    out, want = frame_attention(q, k, v, variant, splits)
    out[0] *= 2.0 ** -power
    want[0] *= 2.0 ** -power
    if splits == 1:
        out[1, :, 5] *= 2.0 ** -power
        want[1, :, 5] *= 2.0 ** -power
    # bf16 probabilities and outputs: each 2^-9 relative, so a value of magnitude <= 4.5 is off by at most 2 * 2^-9 * 4.5
    assert (out - want).abs().max() <= 2e-2


@pytest.mark.parametrize("variant,splits", [(0, 1), (1, 2), (2, 1), (3, 2)])
@pytest.mark.parametrize("rise", [12.0, 20.0, 30.0])
def test_huge_values_whose_weights_rise_along_the_keys(variant, splits, rise):
    """Values of 2^120 and keys `rise` powers of two above those of the first tile: weights times values, at the scale of the first
    tile's weights, are beyond fp32, the output is not."""
    n, H = 64 * 8 + 17, 2
    g = torch.Generator().manual_seed(int(rise) + variant)
    q = 0.25 * torch.randn((H, n, 64), generator=g)
    q[:, :, 0] = 8.0
    k = 0.5 * torch.randn((H, n, 64), generator=g)
    k[:, :, 0] = 0.0
    k[:, 64:, 0] = rise / (8.0 * 0.125 * 1.4426950408889634)
    v = torch.randn((H, n, 64), generator=g) * 2.0 ** 120
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    out, want = frame_attention(q, k, v, variant, splits)
    # bf16 probabilities and outputs: each 2^-9 relative, so a value of magnitude <= 4.5 is off by at most 2 * 2^-9 * 4.5
    assert ((out - want) * 2.0 ** -120).abs().max() <= 2e-2


@pytest.mark.parametrize("variant", [0, 3])
def test_one_infinite_value_leaves_the_other_channels_of_a_cut_row(variant):
    n, H = 64 * 8 + 17, 2
    g = torch.Generator().manual_seed(11)
    q, k, v = (torch.randn((H, n, 64), generator=g).to(torch.bfloat16) for _ in range(3))
    v[0, 30, 7] = float("inf")
    out, want = frame_attention(q, k, v, variant, 2)
    assert torch.equal(out.isinf(), want.isinf()) and int(want.isinf().sum()) == n
    # bf16 probabilities and outputs: each 2^-9 relative, so a value of magnitude <= 4.5 is off by at most 2 * 2^-9 * 4.5
    assert (out - want)[want.isfinite()].abs().max() <= 2e-2


@pytest.mark.parametrize("variant", [0, 1, 2, 3])
@pytest.mark.parametrize("jump", [31.0, 33.0, 127.0, 134.0, 137.0, 300.0])
def test_frame_attention_at_the_limits_of_the_softmax_reference(variant, jump):
    """Around what a reference stands (32 powers of two above the first keys), what one tile may add before it moves (135) and
    beyond."""
    test_frame_attention_when_the_softmax_reference_has_to_move(variant, jump)


@pytest.mark.parametrize("variant", [0, 3])
@pytest.mark.parametrize("rise", [26.0, 28.0, 31.0])
def test_sums_that_move_the_softmax_reference_without_a_large_logit(variant, rise):
    """All keys behind the first tile `rise` powers of two above those of the first: no single probability passes the limit, the
    sum of a few tiles does - for every other query row."""
    n, H = 64 * 8 + 17, 2
    g = torch.Generator().manual_seed(int(rise))
    q = torch.zeros((H, n, 64))
    q[:, ::2, 0] = 8.0
    q[:, :, 1:] = 0.25 * torch.randn((H, n, 63), generator=g)
    k = 0.5 * torch.randn((H, n, 64), generator=g)
    k[:, :, 0] = 0.0
    k[:, 64:, 0] = rise / (8.0 * 0.125 * 1.4426950408889634)
    v = torch.randn((H, n, 64), generator=g)
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    out, want = frame_attention(q, k, v, variant, 1)
    # bf16 probabilities and outputs: each 2^-9 relative, so a value of magnitude <= 4.5 is off by at most 2 * 2^-9 * 4.5
    assert (out - want).abs().max() <= 2e-2


def test_measured_peaks_are_plausible():
    """The library's two yardsticks: an MFMA-only loop and a streaming copy, against the published peaks."""
    mfma, copy = xsv.measure_peaks()
    print(f"measured: MFMA loop {mfma:.0f} TFLOP/s, copy {copy:.0f} GB/s", flush=True)
    assert 800.0 < mfma < 2600.0
    assert 1500.0 < copy < 8200.0


@pytest.mark.parametrize("first,second", [(1, 1), (63, 1), (64, 64), (65, 1), (65, 15), (65, 16), (65, 17), (31, 31), (32, 1), (32, 32), (33, 1), (33, 16), (33, 17), (400, 16), (400, 65), (200, 200)])
@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("P", [900, 4096, 4097, 9000])
def test_topk_where_the_last_candidates_are_compared_with_each_other(first, second, ties, P):
    """`first` scores share the threshold's first digit (11 bits), `second` of them its second: the edges at which the passes of the
    radix select give way to a comparison of all candidates, for lists of one and of several segments and both register counts.  The
    list is whole numbers: equal to that of a stable sort."""
    g = torch.Generator().manual_seed(first * 1000 + second)
    low = (P - first) // 2
    near = (torch.arange(second) if not ties else torch.randint(0, 3, (second,), generator=g)).float() * 2.0 ** -23    # 22 bits alike
    rest = torch.linspace(0.01, 0.2, first - second)                                                                # 11 bits alike
    scores = torch.cat([torch.linspace(0.1, 0.9, low), 1.0 + near, 1.0 + rest, torch.linspace(2.0, 9.0, P - first - low)])
    scores = scores[torch.randperm(P, generator=g)].contiguous()
    order = torch.argsort(scores, descending=True, stable=True)
    above = P - first - low + (first - second)
    for k in sorted({above + 1, above + (second + 1) // 2, above + second}):
        want = torch.sort(order[:k]).values + 7
        keep = xsv.topk_keep(scores.to(DEV), k, 7, 5).cpu().long()
        assert torch.equal(keep[:7], torch.arange(7)) and torch.equal(keep[7:7 + k], want), (first, second, ties, P, k)
        assert torch.equal(keep[7 + k:], 7 + P + torch.arange(5))
