"""The compressor's kinds of tile against the oracle, at the sizes where one gives way to the next.
Every output byte is compared.  Quantizer: arXiv 2206.11357 App. A.4, per group (Sec. 5)."""
import numpy as np
import pytest
import torch

import oracle

import synthetic_inputs as syn
from test_gpu_parity import run_case, to_device, to_host

pytestmark = pytest.mark.gpu


def as_dtype(x, dtype):
    return syn.f32_to_bf16_bits(x) if dtype == "bf16" else x


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("lanes", [k for k in range(3, 32) if k & (k - 1)])
def test_full_tiles_of_group_sizes_that_are_no_power_of_two(gact, dtype, lanes):
    """`lanes` lanes of 32 elements a group.  A last tile that is exactly full, one element short, one
    element long, one group short; the packed string's pad words after each."""
    G = 32 * lanes
    tile = 64 // lanes * G
    for k, n in enumerate((5 * tile, 5 * tile - 1, 5 * tile + 1, 9 * tile - G, tile)):
        x = as_dtype(syn.draw_numpy(syn.OUTLIER, n, 40 * lanes + k), dtype)
        for bits in (1, 2, 4, 8)[(k + lanes) % 2::2]:
            run_case(gact, x, G, bits, seed=lanes + k)


@pytest.mark.parametrize("dtype,bits,blocks", [("bf16", 4, 8192 + 37), ("f32", 2, 8192), ("f32", 1, 16384 + 300),
                                               ("bf16", 2, 32768 + 513), ("f32", 1, 65536 + 1025), ("bf16", 1, 131072 + 2049)])
def test_runs_of_neighbouring_blocks_per_xcd(gact, dtype, bits, blocks):
    """Launches that are long enough for another block order, with and without a last partial window,
    against the same tensor in pieces that are not.  Compress: runs of 16, 32, 64, 128 and 256 blocks;
    decompress: runs of 32."""
    G, seed, n = 256, 9, blocks * 8192 - 1234
    gen = torch.Generator(device="cuda").manual_seed(blocks)
    x = torch.randn(n, device="cuda", generator=gen).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    whole = gact.gact_compress(x, G, bits, seed)
    y = gact.gact_decompress(*whole, n, G, bits, dtype=x.dtype)
    step = 500 * 8192
    ws = torch.empty(gact.gact_multi_workspace_bytes(1), dtype=torch.uint8, device="cuda")
    for a in range(0, n, step):
        m = min(step, n - a)
        p, mn, sc = gact.alloc_compressed(m, G, bits, "cuda")
        descs = gact.make_descs([x[a:a + m]], [p], [mn], [sc], [None], [m], [bits], [seed], [x.dtype], index_bases=[a])
        gact.gact_compress_multi(descs, 1, G, ws)
        assert torch.equal(p, whole[0][a * bits // 8:a * bits // 8 + p.numel()]), a
        assert torch.equal(mn, whole[1][a // G:a // G + mn.numel()]) and torch.equal(sc, whole[2][a // G:a // G + sc.numel()]), a
        assert torch.equal(gact.gact_decompress(p, mn, sc, m, G, bits, dtype=x.dtype).view(torch.uint8),
                           y[a:a + m].view(torch.uint8)), a


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
def test_noise_across_a_wrap_of_the_low_counter_word(gact, dtype):
    """Tiles before, at and after the point where the low word of the Philox block number wraps."""
    G, bits, seed, n = 32, 4, 5, 9 * 2048 + 31
    x = as_dtype(syn.draw_numpy(syn.NORMAL, n, 3), dtype)
    xd = to_device(x)
    for blocks_before in (256, 252, 260, 1024, 4, 508):
        base = 8 * (2**32 - blocks_before)
        p, mn, sc = gact.alloc_compressed(n, G, bits, "cuda")
        descs = gact.make_descs([xd], [p], [mn], [sc], [None], [n], [bits], [seed], [xd.dtype], index_bases=[base])
        gact.gact_compress_multi(descs, 1, G, torch.empty(gact.gact_multi_workspace_bytes(1), dtype=torch.uint8, device="cuda"))
        p_ref, mn_ref, _ = oracle.compress_slice(x, G, bits, seed, base)
        assert np.array_equal(to_host(p), p_ref), blocks_before
        assert np.array_equal(to_host(mn).view(np.uint32), mn_ref.view(np.uint32)), blocks_before


def test_one_launch_of_both_types_and_one_of_each(gact):
    """A launch with fp32 tensors in it and one of bf16 alone are two kernels: the same bytes from both."""
    G, seed = 128, 11
    xs = [to_device(as_dtype(syn.draw_numpy(syn.RELU, n, n), d)) for n, d in
          ((6000, "bf16"), (8192 + 7, "f32"), (4096, "bf16"), (2048 * 5, "f32"), (1, "bf16"))]
    ws = torch.empty(gact.gact_multi_workspace_bytes(len(xs)), dtype=torch.uint8, device="cuda")

    def launch(which, bits):
        out = [gact.alloc_compressed(x.numel(), G, bits, "cuda") for x in which]
        L = len(which)
        descs = gact.make_descs(which, [o[0] for o in out], [o[1] for o in out], [o[2] for o in out], [None] * L,
                                [x.numel() for x in which], [bits] * L, [seed] * L, [x.dtype for x in which])
        gact.gact_compress_multi(descs, L, G, ws)
        return {x.data_ptr(): o for x, o in zip(which, out)}
    for bits in (1, 2, 4, 8):
        both = launch(xs, bits)
        for dt in (torch.float32, torch.bfloat16):
            for ptr, out in launch([x for x in xs if x.dtype == dt], bits).items():
                assert all(torch.equal(a, b) for a, b in zip(out, both[ptr])), (bits, dt)


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("bits", (1, 2, 4, 8))
def test_every_code_in_every_place_of_a_word(gact, dtype, bits):
    """Values on the quantizer's grid: each code at each place of a packed word, and values between
    them, in full tiles and in a last one that ends inside a word."""
    B, G = 2**bits - 1, 64
    rng = np.random.default_rng(bits)
    codes = rng.integers(0, B + 1, size=(64 * 2048) // G * G + 37).astype(np.float32)
    codes[::G], codes[1::G] = 0.0, float(B)            # the group's range: a step of one
    run_case(gact, as_dtype(codes, dtype), G, bits, seed=1)
    run_case(gact, as_dtype(codes + rng.random(codes.size, dtype=np.float32) * np.float32(0.5), dtype), G, bits, seed=2)


def test_steps_are_correctly_rounded(gact):
    """range / (2^b - 1) for ranges of many significands and exponents, down to the smallest that has a step."""
    rng = np.random.default_rng(4)
    G = 32
    expo = np.concatenate([rng.integers(-99, 126, 4000), np.full(500, -100), np.full(500, 126)])
    top = np.ldexp(1.0 + rng.random(expo.size), expo).astype(np.float32)
    x = np.zeros((expo.size, G), dtype=np.float32)
    x[:, 5] = top
    for bits in (1, 2, 4, 8):
        run_case(gact, x.ravel(), G, bits, seed=bits)


def table_bytes(L, blocks):
    """Launch table of L tensors: 56 bytes each, the first block of each and the total, an index over the blocks
    (a power of two of at least 4 L buckets, as few blocks to each as fill no more)."""
    up = lambda v: (v + 15) // 16 * 16
    buckets, shift = 64, 0
    while buckets < 4 * L:
        buckets *= 2
    while (blocks - 1 >> shift) + 1 > buckets:
        shift += 1
    return up(56 * L) + up(4 * (L + 1)) + 4 * ((blocks - 1 >> shift) + 2)


@pytest.mark.parametrize("L,per,copies", [(65, 1, 1), (255, 1, 1), (256, 1, 2), (511, 1, 2), (512, 1, 3), (767, 1, 3),
                                          (768, 1, 0), (600, 5, 3), (620, 6, 0)])
def test_tables_uploaded_in_one_piece_and_in_several(gact, L, per, copies):
    """Launch tables on either side of 16, 32 and 48 KB: one copy of up to 16 KB, two or three of them, one larger
    copy (0).  L tensors of `per` blocks; each tensor's bytes against the call for it alone."""
    size = table_bytes(L, L * per)
    assert copies == (0 if size > 3 * 16384 else -(-size // 16384))
    G, seed, span = 64, 3, 512 if per == 1 else per * 8192
    x = torch.randn(L * span, device="cuda", generator=torch.Generator("cuda").manual_seed(L)).to(torch.bfloat16)
    xs = [x[l * span:l * span + (1 + (l * 37) % 512 if per == 1 else span - l % 9)] for l in range(L)]
    bits = [(1, 2, 4, 8)[l % 4] for l in range(L)]
    bufs = [gact.alloc_compressed(v.numel(), G, b, "cuda") for v, b in zip(xs, bits)]
    ys = [torch.empty_like(v) for v in xs]
    descs = gact.make_descs(xs, [b[0] for b in bufs], [b[1] for b in bufs], [b[2] for b in bufs], ys,
                            [v.numel() for v in xs], bits, [seed + l for l in range(L)], [v.dtype for v in xs])
    ws = torch.empty(gact.gact_multi_workspace_bytes(L), dtype=torch.uint8, device="cuda")
    gact.gact_compress_multi(descs, L, G, ws)
    gact.gact_decompress_multi(descs, L, G, ws)
    for l, (v, b) in enumerate(zip(xs, bits)):
        alone = gact.gact_compress(v, G, b, seed + l)
        assert all(torch.equal(p, q) for p, q in zip(alone, bufs[l])), l
        assert torch.equal(gact.gact_decompress(*alone, v.numel(), G, b, dtype=v.dtype), ys[l]), l


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("G", (32, 96, 128, 704, 1024))
def test_last_tiles_that_end_anywhere(gact, dtype, G):
    """The last tile with 1 to 17 elements, around whole 16-byte pieces, groups, lanes and the tile's end,
    alone and behind a full tile."""
    lanes = G // 32
    tile = 64 // lanes * G
    ends = (1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, G - 1, G, G + 1, tile - 9, tile - 8, tile - 7, tile - 4, tile - 1)
    for k, m in enumerate(ends):
        n = m + tile * (k % 2)
        x = as_dtype(syn.draw_numpy(syn.NORMAL, n, 7 * G + k) + np.float32(3), dtype)
        run_case(gact, x, G, (1, 2, 4, 8)[(k + lanes) % 4], seed=k)


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("bits", (1, 2, 4, 8))
def test_last_blocks_of_the_decompressor(gact, dtype, bits):
    """24,576 elements are whole blocks for every block length in use (2048 to 8192): a last block that is
    full, one element short, one element long, alone and in a launch of several tensors."""
    G, ns = 128, (24576, 24575, 24577, 1, 2 * 24576)
    for k, n in enumerate(ns):
        run_case(gact, as_dtype(syn.draw_numpy(syn.NORMAL, n, 60 + k), dtype), G, bits, seed=k)
    xs = [to_device(as_dtype(syn.draw_numpy(syn.NORMAL, n, 60 + k), dtype)) for k, n in enumerate(ns)]
    bufs = [gact.gact_compress(x, G, bits, k) for k, x in enumerate(xs)]
    ys = [torch.zeros_like(x) for x in xs]
    descs = gact.make_descs(xs, [b[0] for b in bufs], [b[1] for b in bufs], [b[2] for b in bufs], ys, ns,
                            [bits] * len(ns), list(range(len(ns))), [x.dtype for x in xs])
    gact.gact_decompress_multi(descs, len(ns), G, torch.empty(gact.gact_multi_workspace_bytes(len(ns)), dtype=torch.uint8,
                                                              device="cuda"))
    for n, b, x, y in zip(ns, bufs, xs, ys):
        assert torch.equal(gact.gact_decompress(*b, n, G, bits, dtype=x.dtype), y), n


@pytest.mark.parametrize("blocks", (8191, 8192))
def test_two_bit_bf16_blocks_of_short_and_long_launches(gact, blocks):
    """Blocks of 8,192 elements in launches shorter than 8,192 blocks of 6,144, of 6,144 from there on: the
    longest of the short and the shortest of the long, as one tensor and as a list, against short launches."""
    G, bits, n = 128, 2, (blocks - 1) * 6144 + 1
    x = torch.randn(n, device="cuda", generator=torch.Generator("cuda").manual_seed(blocks)).to(torch.bfloat16)
    p, mn, sc = gact.gact_compress(x, G, bits, 3)
    y = gact.gact_decompress(p, mn, sc, n, G, bits, dtype=x.dtype)
    cuts = [k * 700 * 8192 for k in range(n // (700 * 8192) + 1)] + [n]
    parts = [(p[a * bits // 8:], mn[a // G:], sc[a // G:], b - a) for a, b in zip(cuts, cuts[1:])]
    ys = [torch.zeros(q[3], dtype=x.dtype, device="cuda") for q in parts]
    L = len(parts)
    descs = gact.make_descs([None] * L, [q[0] for q in parts], [q[1] for q in parts], [q[2] for q in parts], ys,
                            [q[3] for q in parts], [bits] * L, [0] * L, [x.dtype] * L)
    gact.gact_decompress_multi(descs, L, G, torch.empty(gact.gact_multi_workspace_bytes(L), dtype=torch.uint8, device="cuda"))
    for a, q, part in zip(cuts, parts, ys):
        alone = gact.gact_decompress(*q, G, bits, dtype=x.dtype)
        assert torch.equal(alone.view(torch.int16), y[a:a + q[3]].view(torch.int16)), a
        assert torch.equal(alone.view(torch.int16), part.view(torch.int16)), a


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("bits", (1, 2, 4, 8))
def test_a_range_that_overflows_has_an_infinite_step(gact, dtype, bits):
    """Outside the contract's inputs, but range / B all the same: an infinite step, in full tiles and in the
    last one, and nothing of it in the neighbouring groups."""
    G, n = 64, 3 * 2048 + 5 * 64
    x = syn.draw_numpy(syn.NORMAL, n, 5)
    wide = (3, 40, 97, 100)                            # 97 and 100 lie in the last tile
    for g in wide:
        x[g * G + 7], x[g * G + 50] = -3e38, 3e38
    x = as_dtype(x, dtype)
    p, mn, sc = (to_host(t) for t in gact.gact_compress(to_device(x), G, bits, 2))
    p_ref, mn_ref, sc_ref = oracle.compress(x, G, bits, 2)
    assert np.isposinf(sc[list(wide)]).all()
    assert np.array_equal(sc, sc_ref) and np.array_equal(mn, mn_ref)
    same = np.ones(n // G, dtype=bool)
    same[list(wide)] = False
    per = G * bits // 8
    assert np.array_equal(p[:n // G * per].reshape(-1, per)[same], p_ref[:n // G * per].reshape(-1, per)[same])


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("bits", (1, 2, 4, 8))
@pytest.mark.parametrize("G", (32, 96, 992))
def test_long_decompressing_launches_against_short_ones(gact, dtype, bits, G):
    """The kernel for launches of 8,192 blocks and more and the one for shorter launches: one tensor that ends
    inside a block, and a list of five that each do, against the call for each of the five."""
    units = {1: 3, 2: 4 if dtype == "f32" else 3, 4: 2, 8: 2}[bits]
    span = 4 * units * (256 if dtype == "f32" else 512)
    n = 8192 * span + 777
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn(n, device="cuda", generator=torch.Generator("cuda").manual_seed(bits * G)).to(dt)
    p, mn, sc = gact.gact_compress(x, G, bits, 3)
    y = gact.gact_decompress(p, mn, sc, n, G, bits, dtype=dt)
    step = n // 5 // (128 * G) * 128 * G              # whole groups, and codes that begin on 16 bytes
    cuts = [0, step, 2 * step, 3 * step, 4 * step, n]
    parts = [(p[a * bits // 8:], mn[a // G:], sc[a // G:], b - a) for a, b in zip(cuts, cuts[1:])]
    ys = [torch.zeros(q[3], dtype=dt, device="cuda") for q in parts]
    descs = gact.make_descs([None] * 5, [q[0] for q in parts], [q[1] for q in parts], [q[2] for q in parts], ys,
                            [q[3] for q in parts], [bits] * 5, [0] * 5, [dt] * 5)
    gact.gact_decompress_multi(descs, 5, G, torch.empty(gact.gact_multi_workspace_bytes(5), dtype=torch.uint8, device="cuda"))
    for a, q, part in zip(cuts, parts, ys):
        alone = gact.gact_decompress(*q, G, bits, dtype=dt).view(torch.uint8)
        assert torch.equal(alone, y[a:a + q[3]].view(torch.uint8)), a
        assert torch.equal(alone, part.view(torch.uint8)), a


@pytest.mark.parametrize("blocks", (32767, 32768, 32769 + 130))
@pytest.mark.parametrize("G,bits,mixed", [(256, 2, False), (96, 4, False), (96, 4, True), (416, 2, False), (1024, 1, True), (32, 8, True)])
def test_long_compressing_launches_in_blocks_of_one_wavefront(gact, G, bits, mixed, blocks):
    """The longest launch with fp32 in blocks of four wavefronts and the shortest in blocks of one (groups of 96 only
    beside bf16), the last tile cut: one tensor, and a list of four of which two may be bf16, against calls for pieces of the same noise."""
    tile = 64 // (G // 32) * G
    n = blocks * 4 * tile - tile // 2 - 5
    x = torch.randn(n, device="cuda", generator=torch.Generator("cuda").manual_seed(blocks))
    p, mn, sc = gact.gact_compress(x, G, bits, 3)
    per = 4001 * 128 * G                               # codes of a piece begin on 16 bytes
    step = -(-n // per // 4) * per
    cuts = list(range(0, n, step)) + [n]
    tensors = [x[a:b] for a, b in zip(cuts, cuts[1:])]
    L = len(tensors)
    if mixed:
        tensors = [t.to(torch.bfloat16) if k % 2 else t for k, t in enumerate(tensors)]
    bufs = [gact.alloc_compressed(t.numel(), G, bits, x.device) for t in tensors]
    descs = gact.make_descs(tensors, [b[0] for b in bufs], [b[1] for b in bufs], [b[2] for b in bufs], [None] * L,
                            [t.numel() for t in tensors], [bits] * L, [3] * L, [t.dtype for t in tensors], cuts[:-1])
    ws = torch.empty(gact.gact_multi_workspace_bytes(L), dtype=torch.uint8, device="cuda")
    gact.gact_compress_multi(descs, L, G, ws)
    for k, (t, a) in enumerate(zip(tensors, cuts)):
        m = t.numel()
        alone = gact.alloc_compressed(m, G, bits, x.device)
        for at in range(0, m, per):                    # short launches
            part = t[at:at + per]
            d = gact.make_descs([part], [alone[0][at * bits // 8:]], [alone[1][at // G:]], [alone[2][at // G:]], [None],
                                [part.numel()], [bits], [3], [t.dtype], [a + at])
            gact.gact_compress_multi(d, 1, G, ws)
        assert all(torch.equal(u, v) for u, v in zip(alone, bufs[k])), (k, "list")
        if t.dtype == torch.float32:
            whole = (p[a * bits // 8:][:alone[0].numel()], mn[a // G:][:alone[1].numel()], sc[a // G:][:alone[2].numel()])
            assert all(torch.equal(u, v) for u, v in zip(alone, whole)), (k, "one tensor")
