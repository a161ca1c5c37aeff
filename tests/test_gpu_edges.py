"""Sizes at which the kernels' tiles, remainders and dispatch rules change, against the CPU oracle through the C ABI:
expert FFNs over chosen numbers of rows per expert, and whole layers at chosen token counts."""
import ctypes
import os
import sys

import numpy as np
import pytest
import torch

import workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def launches(call):
    """How many kernels `call` launches: the nodes of a graph that captures it (it has run before)."""
    hip = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
    hip.hipGraphGetNodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    n = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(g.raw_cuda_graph(), None, ctypes.byref(n)) == 0
    return n.value


def placed(a, at):
    """The tensor `a`, or a copy of it that starts `at` elements into its allocation."""
    if at == 0:
        return a
    flat = torch.empty(a.numel() + at, dtype=a.dtype, device=a.device)
    flat[at:] = a.flatten()
    return flat[at:].view(a.shape)


def ffn_rows(moe, rows, d, f, dtype, activation="relu", biases=False, seed=0, mask=None, at=0):
    """moe_expert_ffn over experts with the given row counts, tokens, weights and results `at` elements into their
    allocations; returns (y, the oracle's y at storage precision)."""
    from paper_2405_18832_amd.device_layer import to_device
    E, A = len(rows), int(sum(rows))
    rng = np.random.default_rng([seed, d, f, E, A])
    draw = lambda shape, s: wl.round_to_storage(rng.standard_normal(shape, dtype=np.float32) * np.float32(s), dtype)
    x, w1, w2 = draw((A, d), 1.0), draw((E, f, d), d ** -0.5), draw((E, d, f), f ** -0.5)
    b1, b2 = (draw((E, f), 0.25), draw((E, d), 0.25)) if biases else (None, None)
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    shape = moe.make_shape(A, d, f, E, 1, dtype, False, {"relu": 0, "gelu": 1}[activation])
    dev = lambda a, dt: None if a is None else to_device(a, dt, "cuda")
    packed = []
    for which, w in ((1, w1), (2, w2)):
        src = dev(w, dtype)
        packed.append(placed(torch.empty_like(src), at))
        moe.moe_pack_weights(shape, which, src, packed[-1])
    y = placed(torch.full((A, d), float("nan"), dtype=torch.float32, device="cuda"), at)
    ws = torch.full((moe.moe_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")
    m = None if mask is None else torch.tensor(mask, dtype=torch.uint8, device="cuda")
    moe.moe_expert_ffn_biased(shape, placed(dev(x, dtype), at), packed[0], dev(b1, "f32"), packed[1], dev(b2, "f32"),
                              torch.from_numpy(offsets).cuda(), m, y, ws)
    torch.cuda.synchronize()
    ref = np.full((A, d), np.nan)
    for e in range(E):
        lo, hi = offsets[e], offsets[e + 1]
        if hi > lo and (mask is None or mask[e]):
            ref[lo:hi] = orc.expert_ffn(x[lo:hi], w1[e], w2[e], "bf16" if dtype == "bf16" else None, activation,
                                        *(() if b1 is None else (b1[e], b2[e])))
    return y.cpu().numpy().astype(np.float64), ref


def check(y, ref, tol):
    assert np.array_equal(np.isnan(y), np.isnan(ref))
    on = ~np.isnan(ref[:, 0])
    err = float(orc.rel_error_rows(y[on], ref[on]).max())
    say(f"[edges] element-wise max {err:.3e} (bar {tol:g})")
    assert err <= tol


# fp32 kernel: row tiles of 1 ... 64 rows (4 fragments of 16) and more, contractions below, at and past a 32-k step, row
# pitches that allow 16-, 8- and 4-byte loads, column counts that are no multiple of 16.  Bar: sums of at most 300 products
# in fp32, each within 300 * 2^-24 = 1.8e-5 of the terms' size in the worst case and about 2^-24 * sqrt(300) = 1e-6 in
# practice.
@pytest.mark.parametrize("d,f", [(4, 5), (20, 36), (31, 33), (32, 64), (66, 258), (130, 300)])
def test_f32_ffn_row_tiles(gpu_lib, d, f):
    say(f"[case] f32 ffn d={d} f={f}")
    check(*ffn_rows(gpu_lib, [1, 16, 0, 17, 33, 64, 65, 130], d, f, "f32", "gelu", biases=True), 1e-5)


# the same from base addresses that are 4, 8 and 12 bytes off a 16-byte line, with row pitches of 16 bytes
@pytest.mark.parametrize("at", [1, 2, 3])
@pytest.mark.parametrize("d,f", [(20, 36), (128, 160)])
def test_f32_ffn_unaligned(gpu_lib, d, f, at):
    say(f"[case] f32 ffn d={d} f={f}, {at} elements off")
    check(*ffn_rows(gpu_lib, [1, 17, 40, 64, 65], d, f, "f32", "gelu", biases=True, at=at), 1e-5)


def test_f32_ffn_few_rows_masked(gpu_lib):
    say("[case] f32 ffn few rows, masked")
    check(*ffn_rows(gpu_lib, [3, 9, 4], 64, 96, "f32", mask=[1, 0, 1]), 1e-5)


# fp32 products in units of 32 columns (three units for every CU and 24 rows per tile at least): contractions of an even and an odd number
# of steps, columns that end inside a unit and inside a wavefront's half of it, row tiles of 1 to 4 fragments; first and second product,
# and second products that store the layer's output (compared with the combine step).  Bar: fp32 sums, 1e-5.
@pytest.mark.parametrize("d,f", [(256, 1484), (288, 1508), (1484, 256), (1524, 288)])
def test_f32_wide_units(gpu_lib, d, f):
    say(f"[case] f32 wide units d={d} f={f}")
    check(*ffn_rows(gpu_lib, [64, 128, 63, 49, 48, 33, 65, 17, 120], d, f, "f32", "gelu", biases=True), 1e-5)


def test_f32_wide_top1_output(gpu_lib):
    test_f32_top1_output(gpu_lib, 700, 1484, 256, 9, True)


# first products of a layer in such units: token rows through a row map, every token on two experts, with and without a mask.  Bar as above.
# Columns, contraction, tokens and experts of these and the next are held to those units by test_dispatch_rules.py.
F32_WIDE_LAYER = dict(T=700, d=288, f=1508, E=9, k=2)


@pytest.mark.parametrize("masked", [False, True])
def test_f32_wide_layer(gpu_lib, masked):
    say(f"[case] f32 layer in wide units, masked {masked}")
    moe, (T, d, f, E, k) = gpu_lib, F32_WIDE_LAYER.values()
    rng = np.random.default_rng(T)
    draw = lambda s, *shape: rng.standard_normal(shape, dtype=np.float32) * np.float32(s)
    x, wg, bg = draw(1, T, d), draw(0.05, E, d), draw(0.5, E)
    w1, b1, w2, b2 = draw(d ** -0.5, E, f, d), draw(0.25, E, f), draw(f ** -0.5, E, d, f), draw(0.25, E, d)
    mask = (np.arange(E) % 3 != 1).astype(np.uint8) if masked else np.ones(E, dtype=np.uint8)
    dev = lambda a: torch.from_numpy(a).cuda()
    shape = moe.make_shape(T, d, f, E, k, "f32", True, 1)
    out, idx, gate = torch.full((T, d), float("nan"), device="cuda"), torch.empty((T, k), dtype=torch.int32, device="cuda"), torch.empty((T, k), device="cuda")
    ws = torch.full((moe.moe_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")
    moe.moe_layer_forward_biased(shape, dev(x), dev(wg), dev(bg), dev(w1), dev(b1), dev(w2), dev(b2), dev(mask) if masked else None, -1, out,
                                 idx, gate, ws=ws)
    torch.cuda.synchronize()
    r = orc.route(x, wg, bg, k, True)
    ok = r["margin"] >= 1e-4
    i, g = idx.cpu().numpy(), gate.cpu().numpy().astype(np.float64)
    assert np.array_equal(i[ok], r["idx"][ok])
    ref = np.zeros((T, d))
    for e in np.flatnonzero(mask):
        t, j = np.nonzero(i == e)
        ref[t] += g[t, j][:, None] * orc.expert_ffn(x[t], w1[e], w2[e], None, "gelu", b1[e], b2[e])
    some = ref.any(axis=1)                                 # tokens with an expert that ran
    check(out.cpu().numpy().astype(np.float64)[some], ref[some], 1e-5)
    assert not out.cpu().numpy()[~some].any()


# rounding of such units, of either product by itself (the other only picks columns): no further from 64 bits than the units of 16
# columns, which take operands that are 4 bytes off a 16-byte line.  Contractions of equal halves, of halves a step apart, and long ones.
# Bar on the rms over 500000 elements and more: as above.
F32_WIDE_ROWS, F32_WIDE_ROUNDING = [640, 640, 592, 177], [(256, 772), (288, 768), (2016, 768)]


@pytest.mark.parametrize("first", [True, False])
@pytest.mark.parametrize("K,N", F32_WIDE_ROUNDING)
def test_f32_wide_rounding(gpu_lib, K, N, first):
    say(f"[case] f32 rounding of wide units K={K} N={N} first {first}")
    moe, rows, E, A = gpu_lib, F32_WIDE_ROWS, len(F32_WIDE_ROWS), sum(F32_WIDE_ROWS)
    d, f = (K, N) if first else (N, K)
    gen = torch.Generator(device="cuda").manual_seed(K)
    new = lambda *s: torch.randn(s, device="cuda", generator=gen)
    pick = lambda n, m: torch.eye(m, device="cuda")[torch.randint(0, m, (n,), device="cuda", generator=gen)].expand(E, n, m).contiguous()
    x = new(A, d)
    w1, w2 = (new(E, f, d), pick(d, f)) if first else (pick(f, d), new(E, d, f))
    offsets = torch.tensor([0] + rows, dtype=torch.int32).cumsum(0, dtype=torch.int32).cuda()
    shape = moe.make_shape(A, d, f, E, 1, "f32", False)
    ws = torch.empty(moe.moe_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    lo = offsets.tolist()
    ref = torch.cat([torch.relu(x[i:j].double() @ w1[e].double().t()) @ w2[e].double().t() for e, (i, j) in enumerate(zip(lo, lo[1:]))])
    rms = []
    for at in (0, 1):
        y = placed(torch.full((A, d), float("nan"), device="cuda"), at)
        moe.moe_expert_ffn(shape, placed(x, at), placed(w1, at), placed(w2, at), offsets, None, y, ws)
        rms.append(float((y.double() - ref).square().mean().sqrt()))
    say(f"[edges] rms error {rms[0]:.4e}, in units of 16 columns {rms[1]:.4e}")
    assert rms[0] <= 1.05 * rms[1]


# fp32 rounding: no further from 64 bits than four interleaved fp32 sums over k mod 4, added in pairs, at contractions that one
# wavefront, two, three and all four of them hold, in equal, nearly equal and unequal shares.  Bar on the rms over 512 d elements: 5 %, several times the scatter of
# such a ratio between two orders of the same length.
@pytest.mark.parametrize("d,f", [(20, 20), (32, 32), (48, 40), (64, 64), (96, 160), (256, 128), (264, 544)])
def test_f32_ffn_rounding(gpu_lib, d, f):
    say(f"[case] f32 ffn rounding d={d} f={f}")
    rows = [16, 32, 48, 64, 96, 256]
    rng = np.random.default_rng([0, d, f, len(rows), sum(rows)])              # as ffn_rows draws them
    draw = lambda shape, s: rng.standard_normal(shape, dtype=np.float32) * np.float32(s)
    x, w1, w2 = draw((sum(rows), d), 1.0), draw((len(rows), f, d), d ** -0.5), draw((len(rows), d, f), f ** -0.5)

    def product(a, b):                                                       # a [m, K], b [N, K]: fp32, fused multiply-adds
        s = np.zeros((4, a.shape[0], b.shape[0]), dtype=np.float32)
        for c in range(a.shape[1]):
            s[c % 4] += a[:, c, None].astype(np.float64) * b[None, :, c]
        return (s[0] + s[1]) + (s[2] + s[3])

    lo = np.concatenate([[0], np.cumsum(rows)])
    four = np.concatenate([product(np.maximum(product(x[i:j], w1[e]), 0), w2[e]) for e, (i, j) in enumerate(zip(lo, lo[1:]))])
    y, ref = ffn_rows(gpu_lib, rows, d, f, "f32")
    err, bar = (float(np.sqrt(np.mean((v - ref) ** 2))) for v in (y, four))
    say(f"[edges] rms error {err:.4e}, four sums {bar:.4e}")
    assert err <= 1.05 * bar


def f32_route_against_oracle(moe, T, d, E, at=0):
    k = 2
    rng = np.random.default_rng([T, d, E])
    x, wg = rng.standard_normal((T, d), dtype=np.float32), rng.standard_normal((E, d), dtype=np.float32)
    b = rng.standard_normal(E, dtype=np.float32)
    shape = moe.make_shape(T, d, 4, E, k, "f32", True)
    idx = torch.empty((T, k), dtype=torch.int32, device="cuda")
    w, margin = torch.empty((T, k), device="cuda"), torch.empty(T, device="cuda")
    counts, offsets = (torch.empty(n, dtype=torch.int32, device="cuda") for n in (E, E + 1))
    ws = torch.empty(moe.moe_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    x_dev, wg_dev = (placed(torch.from_numpy(a).cuda(), at) for a in (x, wg))
    moe.moe_route(shape, x_dev, wg_dev, torch.from_numpy(b).cuda(), idx, w, margin, counts, offsets, -1, None, ws)
    torch.cuda.synchronize()
    r = orc.route(x, wg, b, k, True)
    ok = r["margin"] >= 1e-4
    assert np.array_equal(idx.cpu().numpy()[ok], r["idx"][ok])
    assert np.allclose(w.cpu().numpy()[ok], r["g"][ok], rtol=2e-4)
    assert np.array_equal(counts.cpu().numpy(), np.bincount(idx.cpu().numpy().ravel(), minlength=E))


# fp32 routing: contraction remainders and expert counts around one fragment of 16
@pytest.mark.parametrize("T,d,E", [(1, 7, 3), (17, 16, 16), (33, 50, 17), (40, 260, 40)])
def test_f32_route(gpu_lib, T, d, E):
    say(f"[case] f32 route T={T} d={d} E={E}")
    f32_route_against_oracle(gpu_lib, T, d, E)


# the same from base addresses that are 4 and 8 bytes off a 16-byte line
@pytest.mark.parametrize("at", [1, 2])
def test_f32_route_unaligned(gpu_lib, at):
    say(f"[case] f32 route, operands {at} elements off")
    f32_route_against_oracle(gpu_lib, 33, 64, 17, at)


def route_against_oracle(moe, T, d, E, k, x_at=0, wg_at=0, seed=0):
    """moe_route in bf16 against the oracle; x and w_gate start `x_at` / `wg_at` elements into their allocations."""
    rng = np.random.default_rng([seed, T, d, E])
    x = wl.round_to_storage(rng.standard_normal((T, d), dtype=np.float32), "bf16")
    wg = wl.round_to_storage(rng.standard_normal((E, d), dtype=np.float32) * np.float32(d ** -0.5), "bf16")
    b = rng.standard_normal(E, dtype=np.float32)

    dev = lambda a, at: placed(torch.from_numpy(a).cuda().to(torch.bfloat16), at)
    shape = moe.make_shape(T, d, 32, E, k, "bf16", True)
    idx = torch.empty((T, k), dtype=torch.int32, device="cuda")
    w, margin = torch.empty((T, k), device="cuda"), torch.empty(T, device="cuda")
    counts, offsets = (torch.empty(n, dtype=torch.int32, device="cuda") for n in (E, E + 1))
    ws = torch.full((moe.moe_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")
    moe.moe_route(shape, dev(x, x_at), dev(wg, wg_at), torch.from_numpy(b).cuda(), idx, w, margin, counts, offsets, -1, None, ws)
    torch.cuda.synchronize()
    r = orc.route(x, wg, b, k, True)
    ok = r["margin"] >= 1e-4
    assert ok.mean() > 0.95
    assert np.array_equal(idx.cpu().numpy()[ok], r["idx"][ok])
    assert np.allclose(w.cpu().numpy()[ok], r["g"][ok], rtol=2e-4)
    assert np.allclose(margin.cpu().numpy(), r["margin"], rtol=0, atol=2e-4)
    assert np.array_equal(counts.cpu().numpy(), np.bincount(idx.cpu().numpy().ravel(), minlength=E))


# bf16 routing: every form of the kernel (16, 32 or 64 tokens by 64 or 128 experts at a time; on 256 CUs 32 tokens from 4097
# tokens on and 64 from 8193), ragged token counts, contractions that go round the ring of four stages of 64 k more than once
# and end in half a stage, one that is half a stage, expert counts that take a second pass, and the few-token path; up to 32
# experts from d = 1024 on, where the wavefronts share the contraction (equally, unequally, with a half stage in the last share),
# and more than 64 tokens per CU
@pytest.mark.parametrize("T,d,E,k", [(65, 1024, 32, 2), (700, 1056, 9, 1), (4100, 1120, 17, 2), (8192, 1184, 3, 2), (8300, 1056, 31, 4),
                                     (17000, 1024, 8, 1), (17000, 160, 40, 2), (65, 352, 60, 2), (700, 320, 129, 4),
                                     (300, 608, 1024, 8), (4100, 352, 60, 2), (5003, 352, 128, 2),
                                     (4500, 352, 200, 3), (8192, 96, 64, 1), (8300, 352, 40, 2), (8300, 544, 128, 2),
                                     (8300, 352, 200, 1), (9000, 32, 20, 2), (33, 352, 60, 2), (64, 96, 300, 2)])
def test_bf16_route(gpu_lib, T, d, E, k):
    say(f"[case] bf16 route T={T} d={d} E={E}")
    route_against_oracle(gpu_lib, T, d, E, k)


# a token whose logits are all NaN: no maximum exists, every slot holds expert 0 and a NaN weight, whatever the number of
# experts (64, 128 and 256 are kept in registers, more are not), and other tokens are as without it
@pytest.mark.parametrize("T,E", [(40, 20), (40, 100), (40, 200), (40, 300), (100, 100), (100, 300)])
def test_nan_token(gpu_lib, T, E):
    say(f"[case] NaN token T={T} E={E}")
    moe, d, k, bad = gpu_lib, 64, 3, 7
    gen = torch.Generator(device="cuda").manual_seed(E)
    x, wg = (torch.randn((n, d), device="cuda", generator=gen).to(torch.bfloat16) for n in (T, E))
    shape = moe.make_shape(T, d, 32, E, k, "bf16", False)
    ws = torch.empty(moe.moe_workspace_bytes(shape), dtype=torch.uint8, device="cuda")

    def route(x):
        idx, w = torch.empty((T, k), dtype=torch.int32, device="cuda"), torch.empty((T, k), device="cuda")
        counts, offsets = (torch.empty(n, dtype=torch.int32, device="cuda") for n in (E, E + 1))
        moe.moe_route(shape, x, wg, None, idx, w, None, counts, offsets, -1, None, ws)
        torch.cuda.synchronize()
        assert torch.equal(counts.cpu().long(), torch.bincount(idx.cpu().flatten().long(), minlength=E))
        return idx, w

    idx, w = route(x)
    x[bad, 5] = float("nan")
    idx2, w2 = route(x)
    assert idx2[bad].tolist() == [0] * k and bool(torch.isnan(w2[bad]).all())
    others = torch.arange(T, device="cuda") != bad
    assert torch.equal(idx[others], idx2[others]) and torch.equal(w[others], w2[others])


# the same from operands that are views into larger buffers, 2, 4 and 8 bytes off a 16-byte line
@pytest.mark.parametrize("x_at,wg_at", [(0, 1), (4, 0), (1, 2)])
@pytest.mark.parametrize("T,d,E,k", [(70, 352, 60, 2), (700, 320, 129, 4), (4100, 352, 60, 2), (5003, 96, 128, 2), (8300, 352, 40, 2),
                                     (8300, 32, 100, 1), (33, 96, 60, 2), (300, 1056, 30, 2), (4100, 1120, 8, 1), (8300, 1056, 12, 2)])
def test_bf16_route_unaligned(gpu_lib, T, d, E, k, x_at, wg_at):
    say(f"[case] bf16 route T={T} d={d} E={E}, operands {x_at} and {wg_at} elements off")
    route_against_oracle(gpu_lib, T, d, E, k, x_at, wg_at)


# layers of few tokens, which are routed inside the first product and combined inside the second (three launches, counted below): one
# assignment up to the most, contractions of an odd number of 32-k steps, of fewer pairs of steps than wavefronts and of many, units
# of 16 columns and of 64 (256 of them, and more than a round), and a token of NaN logits, whose slots all name expert 0 and, with 8 of
# them, give it more rows than a tile holds.  The last four are layers of few tokens that the general path is faster for.  Values against
# the oracle at storage precision; bar: the output's one rounding to bf16 (2^-8) and rare hidden values at a rounding boundary.  Routing
# and places also against the general path, which a mask of ones takes, and its output within the same bar.
@pytest.mark.parametrize("nan_token", [False, True])
@pytest.mark.parametrize("T,d,f,E,k,few", [(1, 32, 32, 1, 1, True), (1, 96, 96, 5, 3, True), (3, 160, 544, 256, 2, True),
                                           (5, 352, 608, 40, 2, True), (7, 2048, 256, 20, 2, True), (2, 64, 1056, 8, 8, True),
                                           (4, 64, 352, 64, 5, True), (4, 1024, 1024, 40, 4, True), (2, 1024, 8192, 3, 1, True),
                                           (8, 1024, 4096, 8, 1, True), (1, 4096, 1120, 6, 4, True),
                                           (8, 64, 1056, 8, 8, False), (2, 64, 8192, 30, 1, False), (8, 64, 1024, 64, 4, False),
                                           (4, 96, 3072, 64, 3, False)])
def test_few_tokens(gpu_lib, T, d, f, E, k, few, nan_token):
    say(f"[case] few tokens T={T} d={d} f={f} E={E} k={k} nan={nan_token}")
    moe = gpu_lib
    from paper_2405_18832_amd.device_layer import to_device
    rng = np.random.default_rng([T, d, f, E, k])
    draw = lambda shape, s: wl.round_to_storage(rng.standard_normal(shape, dtype=np.float32) * np.float32(s), "bf16")
    x, wg, w1, w2 = draw((T, d), 1.0), draw((E, d), d ** -0.5), draw((E, f, d), d ** -0.5), draw((E, d, f), f ** -0.5)
    bg, b1, b2 = draw((E,), 0.5), draw((E, f), 0.25), draw((E, d), 0.25)
    bad = T // 2 if nan_token else -1
    if nan_token:
        x[bad, d // 2] = np.nan
    act = "gelu" if T % 2 else "relu"
    shape = moe.make_shape(T, d, f, E, k, "bf16", True, {"relu": 0, "gelu": 1}[act])
    dev = lambda a, dt: to_device(a, dt, "cuda")
    xd, wgd, bgd, b1d, b2d = dev(x, "bf16"), dev(wg, "bf16"), dev(bg, "f32"), dev(b1, "f32"), dev(b2, "f32")
    p1, p2 = torch.empty((E, d * f), dtype=torch.bfloat16, device="cuda"), torch.empty((E, d * f), dtype=torch.bfloat16, device="cuda")
    moe.moe_pack_weights(shape, 1, dev(w1, "bf16"), p1)
    moe.moe_pack_weights(shape, 2, dev(w2, "bf16"), p2)
    ws = torch.full((moe.moe_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")

    def layer(mask, by_products=True):
        out = torch.full((T, d), 7.0, dtype=torch.bfloat16, device="cuda")
        i32 = lambda *s: torch.full(s, -1, dtype=torch.int32, device="cuda")
        more = (i32(T, k), torch.zeros((T, k), device="cuda"), i32(E), i32(T * k), torch.zeros(E, dtype=torch.uint8, device="cuda"))
        moe.moe_layer_forward_biased(shape, xd, wgd, bgd, p1, b1d, p2, b2d, mask, -1, out, *(more if by_products else (None,) * 5), ws=ws)
        torch.cuda.synchronize()
        return out, more

    out, by = layer(None)
    general, gen = layer(torch.ones(E, dtype=torch.uint8, device="cuda"))
    scratch = torch.empty_like(out)
    n = launches(lambda: moe.moe_layer_forward_biased(shape, xd, wgd, bgd, p1, b1d, p2, b2d, None, -1, scratch, ws=ws))
    assert (n == 3) == few, n
    others = np.arange(T) != bad
    for a, b in zip(by, gen):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    if others.any():
        a, b = (t.float().cpu().numpy().astype(np.float64)[others] for t in (out, general))
        assert float(orc.rel_error_rows(a, b).max()) <= 1e-2
    bare, _ = layer(None, by_products=False)               # none of the optional outputs
    assert torch.equal(bare.view(torch.int16), out.view(torch.int16))
    idx, g = by[0].cpu().numpy(), by[1].cpu().numpy().astype(np.float64)
    r = orc.route(np.where(np.isnan(x), 0, x), wg, bg, k, True)
    ok = others & (r["margin"] >= 1e-4)
    assert np.array_equal(idx[ok], r["idx"][ok])
    ref = np.zeros((T, d))
    for t in np.flatnonzero(others):
        for j in range(k):
            e = idx[t, j]
            ref[t] += g[t, j] * orc.expert_ffn(x[t:t + 1], w1[e], w2[e], "bf16", act, b1[e], b2[e])[0]
    got = out.float().cpu().numpy().astype(np.float64)
    if others.any():
        err = float(orc.rel_error_rows(got[others], ref[others]).max())
        say(f"[edges] element-wise max {err:.3e}")
        assert err <= 1e-2
    assert not nan_token or np.isnan(got[bad]).all()


# tiled kernels: experts around their 128- and 256-row tiles, columns that are no multiple of a tile's, contractions of one
# step, of fewer steps than the LDS ring holds, and long enough to be cut; the last shape has few large units in one product
# and many in the other.  Bar: y against the oracle that rounds the hidden activation once, as the kernels do; what is left
# is fp32 sums (2^-24 * sqrt(K) of the terms) and a rare hidden value at a rounding boundary (2^-8 of one of f terms).
@pytest.mark.parametrize("d,f", [(32, 96), (96, 160), (160, 1056), (64, 5120)])
def test_tiled_ffn_row_tiles(gpu_lib, d, f):
    say(f"[case] tiled ffn d={d} f={f}")
    check(*ffn_rows(gpu_lib, [128, 129, 64, 255, 0, 257, 300, 1], d, f, "bf16", "gelu", biases=True), 4e-3)


# experts of 65 ... 127 rows next to a large one: as many as join the tiled kernel (256 CUs: 8 half-sized tiles at 4096 columns)
# and one more, which leaves them to the streaming kernel; and products just inside and outside one round of the tiled kernel's
# 128 x 128 units, and of its 256 x 128 units, with contractions shorter than the ring and longer than 96 steps.  Bar as above.
@pytest.mark.parametrize("act", ["relu", "gelu"])
@pytest.mark.parametrize("rows,d,f", [([128] + 7 * [100], 64, 4096), ([128] + 8 * [100], 64, 4096), ([256] + 6 * [65, 0], 4096, 32),
                                      (8 * [129], 64, 2048), (8 * [129] + [128], 64, 2048), (15 * [256], 96, 2048),
                                      (16 * [130], 96, 2048), (17 * [129], 1024, 160), (22 * [130], 1024, 3104)])
def test_unit_choice(gpu_lib, rows, d, f, act):
    say(f"[case] unit choice {len(rows)} experts d={d} f={f} {act}")
    check(*ffn_rows(gpu_lib, rows, d, f, "bf16", act, biases=True), 4e-3)


# one kernel per product for large and small experts: streaming units alone, in more rounds than one, with contractions of an odd number
# of steps from rows in LDS (up to all 128 KiB) and split over two and four wavefronts; fine units cut into 3, 5, 7 and 8 parts (48, 72, ...
# steps), with no streaming units, with a few and with more than there are blocks; big units left over after full rounds, whole (contractions of 8
# and 9 steps), cut in two and in three, the last columns of a unit missing.  Row tiles of 1 to 4 fragments, and of 1 and 64 rows.  Bar as above.
# Last item of a case: units, full rounds, units left over and parts of each, of the two products (test_dispatch_rules.py holds them to that).
SMALL_ROWS = [1, 16, 17, 32, 33, 48, 49, 64, 63]
PRODUCT_UNITS = [(SMALL_ROWS, 992, 1056, None), (5 * SMALL_ROWS, 96, 3104, None), (SMALL_ROWS, 1056, 96, None),
                 ([130], 64, 2304, [("fine", 0, 36, 1), ("fine", 0, 2, 3)]),
                 ([130] + SMALL_ROWS, 64, 3840, [("fine", 0, 60, 1), ("fine", 0, 2, 5)]),
                 ([129, 200] + SMALL_ROWS, 96, 5376, [("fine", 0, 168, 1), ("fine", 0, 4, 7)]),
                 ([130] + 12 * SMALL_ROWS, 160, 6144, [("fine", 0, 96, 1), ("fine", 0, 4, 8)]),
                 ([2400] + SMALL_ROWS, 256, 7168, [("big", 1, 24, 1), ("fine", 0, 38, 6)]),
                 ([2400] + 4 * SMALL_ROWS, 288, 7200, [("big", 1, 34, 1), ("fine", 0, 57, 4)]),
                 (9 * [256] + SMALL_ROWS, 2048, 288, [("fine", 0, 54, 2), ("narrow", 0, 144, 1)]),
                 ([8700] + SMALL_ROWS, 2112, 2048, [("big", 1, 16, 2), ("big", 1, 50, 2)]),
                 ([33000] + SMALL_ROWS, 512, 3072, [("big", 6, 12, 1), ("big", 1, 2, 3)])]


@pytest.mark.parametrize("rows,d,f", [case[:3] for case in PRODUCT_UNITS])
def test_product_units(gpu_lib, rows, d, f):
    say(f"[case] product units {len(rows)} experts, largest {max(rows)} rows, d={d} f={f}")
    check(*ffn_rows(gpu_lib, rows, d, f, "bf16", "relu", biases=True), 4e-3)


def ffn_on_device(moe, rows, x, w1, w2, act="relu"):
    """fp32 rows of moe_expert_ffn over bf16 tensors: x [A, d], w1 [E, f, d], w2 [E, d, f]."""
    E, f, d = w1.shape
    shape = moe.make_shape(sum(rows), d, f, E, 1, "bf16", False, {"relu": 0, "gelu": 1}[act])
    p1, p2 = torch.empty_like(w1), torch.empty_like(w2)
    moe.moe_pack_weights(shape, 1, w1.contiguous(), p1)
    moe.moe_pack_weights(shape, 2, w2.contiguous(), p2)
    offsets = torch.tensor([0] + list(rows), dtype=torch.int32).cumsum(0, dtype=torch.int32).cuda()
    y = torch.full((sum(rows), d), float("nan"), device="cuda")
    ws = torch.full((moe.moe_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")
    moe.moe_expert_ffn(shape, x.contiguous(), p1, p2, offsets, None, y, ws)
    torch.cuda.synchronize()
    return y


# The rows of a large expert are the same sums whether or not there are small experts to stream: 34 x 8 units, 16 of which are left over
# after a full round and cut in two.  The second product only picks columns of h.
def test_cut_units_beside_streaming(gpu_lib):
    say("[case] cut units beside streaming units")
    d, f, m, small = 2048, 2048, 34 * 256, 50
    gen = torch.Generator(device="cuda").manual_seed(m)
    x = torch.randn((m + small * 64, d), device="cuda", generator=gen).to(torch.bfloat16)
    w1 = (torch.randn((1 + small, f, d), device="cuda", generator=gen) * d ** -0.5).to(torch.bfloat16)
    w2 = torch.eye(f, device="cuda", dtype=torch.bfloat16)[torch.randperm(f, device="cuda", generator=gen)[:d]].expand(1 + small, d, f)
    alone = ffn_on_device(gpu_lib, [m], x[:m], w1[:1], w2[:1])
    beside = ffn_on_device(gpu_lib, [m] + small * [64], x, w1, w2)
    assert torch.equal(beside[:m], alone)


# 256 x 128 units add a contraction up in as many partial sums as full-width units would have been cut into (none is longer than
# those): their rows are the fp32 sums, in order, of calls over a run of 32 steps each, bit for bit.  Integers that the first product
# adds up exactly make h the same in all calls.
@pytest.mark.parametrize("E,m,d,runs", [(9, 256, 2048, 2), (10, 250, 2048, 3), (14, 256, 2048, 2)])
def test_narrow_units_partial_sums(gpu_lib, E, m, d, runs):
    say(f"[case] partial sums of narrow units, {E} x {m} rows d={d}, {runs} runs")
    gen = torch.Generator(device="cuda").manual_seed(E * m)
    whole = lambda lo, hi, *s: torch.randint(lo, hi, s, device="cuda", generator=gen).to(torch.bfloat16)
    f = 1024 * runs
    x, w1 = whole(-2, 3, E * m, d), whole(-1, 2, E, f, d)
    w2 = (torch.randn((E, d, f), device="cuda", generator=gen) * f ** -0.5).to(torch.bfloat16)
    y = ffn_on_device(gpu_lib, E * [m], x, w1, w2)
    parts = [ffn_on_device(gpu_lib, E * [m], x, w1[:, i:i + 1024], w2[:, :, i:i + 1024]) for i in range(0, f, 1024)]
    want = parts[0]
    for p in parts[1:]:
        want = want + p
    assert torch.equal(y, want)


# GeLU: the first product of all experts at once (256 x 128 units) and of two experts at a time (128 x 128 units, each two halves of the
# contraction) round the same sums.  The second product only picks columns of h.
@pytest.mark.parametrize("m,d", [(256, 768), (188, 1024)])
def test_narrow_units_gelu_sums(gpu_lib, m, d):
    say(f"[case] GeLU sums of narrow units, {m} rows d={d}")
    E, f = 24, 1024
    gen = torch.Generator(device="cuda").manual_seed(m)
    x = torch.randn((E * m, d), device="cuda", generator=gen).to(torch.bfloat16)
    w1 = (torch.randn((E, f, d), device="cuda", generator=gen) * d ** -0.5).to(torch.bfloat16)
    w2 = torch.eye(f, device="cuda", dtype=torch.bfloat16)[torch.randperm(f, device="cuda", generator=gen)[:d]].expand(E, d, f)
    y = ffn_on_device(gpu_lib, E * [m], x, w1, w2, "gelu")
    two = [ffn_on_device(gpu_lib, 2 * [m], x[e * m:(e + 2) * m], w1[e:e + 2], w2[e:e + 2], "gelu") for e in range(0, E, 2)]
    assert torch.equal(y, torch.cat(two))


# counting sort: one block, a block per 16 or 4 chunks, and slot bases through memory, at the sizes where one form gives way to
# the next (4096 assignments for moe_permute; 256 experts; 64 k histogram entries or 1024 chunks), by itself and in the layer.
# Past 64 k entries: the layer with chunks of 16 tokens and 257 experts, moe_permute with chunks of 256 assignments and 1024
# experts (placed from the caller's offsets).  70000 x 3 makes 1094 chunks in the layer.
@pytest.mark.parametrize("T,E,k", [(1, 1, 1), (64, 256, 8), (64, 257, 2), (65, 256, 8), (2048, 40, 2), (2049, 40, 2),
                                   (4000, 257, 3), (4080, 257, 1), (4096, 256, 1), (4100, 257, 1), (4112, 256, 1), (5000, 1024, 2),
                                   (16384, 1024, 1), (16641, 1024, 1), (70000, 3, 1)])
def test_places(gpu_lib, T, E, k):
    say(f"[case] places T={T} E={E} k={k}")
    moe, d = gpu_lib, 32
    gen = torch.Generator(device="cuda").manual_seed(T + E)
    bf = lambda *s: torch.randn(s, device="cuda", generator=gen).to(torch.bfloat16)
    i32 = lambda *s: torch.full(s, -1, dtype=torch.int32, device="cuda")
    x, wg, w = bf(T, d), bf(E, d), bf(E, d * d)
    shape = moe.make_shape(T, d, d, E, k, "bf16", True)
    ws = torch.full((moe.moe_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")
    out, gate = torch.empty((T, d), dtype=torch.bfloat16, device="cuda"), torch.empty((T, k), device="cuda")
    got = []
    idx, counts, perm = i32(T, k), i32(E), i32(T * k)
    mask = torch.empty(E, dtype=torch.uint8, device="cuda")
    moe.moe_layer_forward(shape, x, wg, None, w, w, None, E // 2, out, idx, gate, counts, perm, mask, ws=ws)
    got.append((idx, counts, perm))
    idx, counts, perm, inv, offsets, xp = i32(T, k), i32(E), i32(T * k), i32(T * k), i32(E + 1), torch.empty_like(bf(T * k, d))
    moe.moe_route(shape, x, wg, None, idx, gate, None, counts, offsets, -1, None, ws)
    moe.moe_permute(shape, x, idx, offsets, perm, inv, xp, ws)
    got.append((idx, counts, perm))
    torch.cuda.synchronize()
    for i, c, p in got:
        flat = i.cpu().numpy().ravel()
        want = np.argsort(flat, kind="stable")
        assert np.array_equal(c.cpu().numpy(), np.bincount(flat, minlength=E))
        assert np.array_equal(p.cpu().numpy(), want)
    n = np.bincount(flat, minlength=E)
    assert np.array_equal(offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(n)]))
    assert np.array_equal(inv.cpu().numpy()[want], np.arange(T * k))
    assert torch.equal(xp.view(torch.int16), x[torch.from_numpy(want // k).cuda()].view(torch.int16))
    assert np.array_equal(mask.cpu().numpy(), orc.hot_mask_top_h(n, E // 2))


# The events of a profiled call time a product's large and small experts apart: 28 us and more of 256 tiled units, 60 us of 335 MB of
# streamed weights per product.  Bar: a tenth of their sum, several times what two events without a unit between them are apart.
# Events [1] and [3] left out: the product's one kernel.  The outputs are the same bits.
def test_profile_events_time_the_kinds_apart(gpu_lib):
    say("[case] profile events of large and small experts")
    moe, d, f, small = gpu_lib, 1024, 4096, 40
    rows = [4096] + small * [64]
    gen = torch.Generator(device="cuda").manual_seed(7)
    bf = lambda s, *shape: (torch.randn(shape, device="cuda", generator=gen) * s).to(torch.bfloat16)
    x, w1, w2 = bf(1.0, sum(rows), d), bf(d ** -0.5, len(rows), f, d), bf(f ** -0.5, len(rows), d, f)
    want = ffn_on_device(moe, rows, x, w1, w2)
    events = [torch.cuda.Event(enable_timing=True) for _ in range(5)]
    for e in events:
        e.record()                                         # creates the handle
    torch.cuda.synchronize()
    for skip in ((), (1, 3)):
        moe.moe_set_profile_events([None if i in skip else e.cuda_event for i, e in enumerate(events)])
        try:
            y = ffn_on_device(moe, rows, x, w1, w2)
        finally:
            moe.moe_set_profile_events(None)
        assert torch.equal(y, want)
        at = [i for i in range(5) if i not in skip]
        us = [1e3 * events[a].elapsed_time(events[b]) for a, b in zip(at, at[1:])]
        say(f"[edges] us between events {at}: {[round(u, 1) for u in us]}")
        assert min(us) >= 0.1 * sum(us)


# hot_mask_out is an output only: once the dispatch step has written it (the profile event before the first product stands
# behind that step), the caller may overwrite it on another stream while the products still run
@pytest.mark.parametrize("T,E,k", [(48, 40, 2), (1500, 24, 2)])
def test_derived_mask_output_is_not_read_back(gpu_lib, T, E, k):
    say(f"[case] derived mask overwritten during the call T={T} E={E}")
    moe, d, f = gpu_lib, 1024, 4096
    gen = torch.Generator(device="cuda").manual_seed(T)
    bf = lambda s, *shape: (torch.randn(shape, device="cuda", generator=gen) * s).to(torch.bfloat16)
    x, wg, w1, w2 = bf(1.0, T, d), bf(0.05, E, d), bf(d ** -0.5, E, d * f), bf(f ** -0.5, E, d * f)
    shape = moe.make_shape(T, d, f, E, k, "bf16", True)
    ws = torch.empty(moe.moe_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    want = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    out, mask = torch.empty_like(want), torch.empty(E, dtype=torch.uint8, device="cuda")
    moe.moe_layer_forward(shape, x, wg, None, w1, w2, None, E // 3, want, ws=ws)
    before_products, other = torch.cuda.Event(), torch.cuda.Stream()
    before_products.record()                               # creates the handle
    torch.cuda.synchronize()
    moe.moe_set_profile_events([before_products.cuda_event, None, None, None, None])
    try:
        moe.moe_layer_forward(shape, x, wg, None, w1, w2, None, E // 3, out, hot_mask_out=mask, ws=ws)
    finally:
        moe.moe_set_profile_events(None)
    other.wait_event(before_products)
    with torch.cuda.stream(other):
        written = mask.clone()
        mask.zero_()
    torch.cuda.synchronize()
    assert int(written.sum()) == E // 3 and int(mask.sum()) == 0
    assert torch.equal(out.view(torch.int16), want.view(torch.int16))


# fp32 layers of one expert per token, whose second product stores the layer's output itself: tiles of 1, 16, 17, 64 and 65 rows,
# the three widths of loads, sums in four, two and one chains, columns that end inside a unit, tokens without numbers; the first six
# with the assignments sorted inside the first product (`sorts`), the others past the limits of that.  An output that is not 16-byte
# aligned is left to combine, as is a layer with a mask of ones: the same sums, one multiply and one rounding, bit for bit.
@pytest.mark.parametrize("T,d,f,E,sorts", [(1, 32, 33, 1, True), (17, 20, 33, 1, True), (64, 64, 96, 1, True), (65, 33, 70, 1, True),
                                           (200, 66, 160, 5, True), (500, 258, 512, 8, True), (300, 33, 71, 65, False),
                                           (330, 34, 70, 66, False), (300, 20, 72, 70, False), (1025, 36, 128, 16, False),
                                           (1000, 66, 1042, 16, False), (900, 33, 1044, 14, False), (950, 130, 2049, 9, False)])
def test_f32_top1_output(gpu_lib, T, d, f, E, sorts):
    say(f"[case] f32 top-1 output T={T} d={d} f={f} E={E}")
    moe = gpu_lib
    gen = torch.Generator(device="cuda").manual_seed(T + d + f)
    new = lambda *s: torch.randn(s, device="cuda", generator=gen)
    x, wg, bg, w1, b1, w2, b2 = new(T, d), new(E, d), new(E), new(E, f, d), new(E, f), new(E, d, f), new(E, d)
    x[T // 2, 0] = float("nan")
    shape = moe.make_shape(T, d, f, E, 1, "f32", False, 1)
    ws = torch.full((moe.moe_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")
    ones = torch.ones(E, dtype=torch.uint8, device="cuda")

    def call(mask, out):
        moe.moe_layer_forward_biased(shape, x, wg, bg, w1, b1, w2, b2, mask, -1, out, ws=ws)

    outs, kernels = [], []
    for mask, at in ((None, 0), (None, 1), (ones, 0), (ones, 1)):
        buf = torch.full((at + T * d + 8,), 7.0, device="cuda")
        call(mask, buf[at:at + T * d].view(T, d))
        torch.cuda.synchronize()
        assert bool((buf[:at] == 7.0).all()) and bool((buf[at + T * d:] == 7.0).all())
        outs.append(torch.where(buf.isnan(), 8.0, buf)[at:at + T * d].view(torch.int32))
        kernels.append(launches(lambda: call(mask, buf[at:at + T * d].view(T, d))))
    for o in outs[1:]:
        assert torch.equal(outs[0], o)
    # with a mask: routing, dispatch, two products, combine; the fold saves the last, sorting the second
    assert kernels == [4 - sorts, 5 - sorts, 5, 5]


# fp32 layers whose first product sorts the assignments: groups of 64 assignments and 256 threads with and without a rest, the most
# assignments and experts and one more (which take the general path), column groups that are and are not a multiple of 8, more units in
# an XCD's slice than its even share, a token of NaN logits whose slots all name expert 0.  The same order and sums as the general
# path, which a mask of ones takes: bit for bit.  Order and values also by themselves: perm is the stable sort of the experts, and
# the output the oracle's; bar of the fp32 FFN tests above.
@pytest.mark.parametrize("T,d,f,E,k,sorts", [(1, 32, 16, 1, 1, True), (64, 64, 256, 8, 2, True), (63, 33, 70, 5, 1, True),
                                             (65, 130, 128, 33, 1, True), (128, 20, 144, 64, 8, True), (129, 64, 32, 8, 8, False),
                                             (128, 64, 32, 8, 8, True), (256, 66, 40, 4, 4, True), (1024, 32, 144, 64, 1, True),
                                             (1025, 32, 64, 64, 1, False), (300, 32, 64, 65, 2, False), (3, 96, 2048, 3, 3, True),
                                             (20, 464, 1312, 8, 2, True), (33, 80, 300, 32, 2, True)])
def test_f32_sort_in_first_product(gpu_lib, T, d, f, E, k, sorts):
    say(f"[case] f32 sort in first product T={T} d={d} f={f} E={E} k={k}")
    moe = gpu_lib
    gen = torch.Generator(device="cuda").manual_seed(T + d + f)
    new = lambda *s: torch.randn(s, device="cuda", generator=gen)
    x, wg, bg, w1, b1, w2, b2 = new(T, d), new(E, d), new(E), new(E, f, d), new(E, f), new(E, d, f), new(E, d)
    x[T // 2, 0] = float("nan")
    shape = moe.make_shape(T, d, f, E, k, "f32", True, 1)
    ws = torch.full((moe.moe_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")
    ones = torch.ones(E, dtype=torch.uint8, device="cuda")

    def layer(mask, by_products=True):
        i32 = lambda *s: torch.full(s, -1, dtype=torch.int32, device="cuda")
        more = (i32(T, k), torch.zeros((T, k), device="cuda"), i32(E), i32(T * k), torch.zeros(E, dtype=torch.uint8, device="cuda"))
        out = torch.full((T, d), 7.0, device="cuda")
        moe.moe_layer_forward_biased(shape, x, wg, bg, w1, b1, w2, b2, mask, -1, out, *(more if by_products else (None,) * 5), ws=ws)
        torch.cuda.synchronize()
        return [torch.where(a.isnan(), 8.0, a) if a.is_floating_point() else a for a in (out, *more)]

    few, general = layer(None), layer(ones)
    for a, b in zip(few, general):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    assert torch.equal(layer(None, by_products=False)[0], few[0])
    scratch = torch.empty_like(few[0])
    kernels = [launches(lambda: moe.moe_layer_forward_biased(shape, x, wg, bg, w1, b1, w2, b2, m, -1, scratch, ws=ws))
               for m in (None, ones)]
    assert kernels == [5 - sorts - (k == 1), 5]
    idx, g = few[1].cpu().numpy(), few[2].cpu().numpy().astype(np.float64)
    assert np.array_equal(few[4].cpu().numpy(), np.argsort(idx.ravel(), kind="stable"))
    assert np.array_equal(few[3].cpu().numpy(), np.bincount(idx.ravel(), minlength=E))
    host = [t.cpu().numpy() for t in (x, w1, w2, b1, b2)]
    ref = np.zeros((T, d))
    for e in range(E):
        t, j = np.nonzero((idx == e) & (np.arange(T) != T // 2)[:, None])
        if len(t):
            ref[t] += g[t, j, None] * orc.expert_ffn(host[0][t], host[1][e], host[2][e], None, "gelu", host[3][e], host[4][e])
    others = np.arange(T) != T // 2
    if others.any():
        assert float(orc.rel_error_rows(few[0].cpu().numpy().astype(np.float64)[others], ref[others]).max()) <= 1e-5
