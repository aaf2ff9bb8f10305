"""The reductions' launch forms at the sizes where one gives way to the next, against the oracle
(arXiv 2206.11357: Alg. 1, the variance alert of Sec. 4.2, the footprint of Sec. 5.2)."""
import numpy as np
import pytest
import torch

import oracle
import synthetic_inputs as syn
from test_gpu_sensitivity import REL, buffers, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
def test_footprint_sums_per_block_and_samples_in_one_kernel(gact, dtype):
    """Sizes around tiles and blocks of the fused call (wavefronts without a tile, group sizes that are no
    power of two), no sample points, one, more than a block of them.  The terms are added in binary64 in
    another order than the oracle's: at most about 60 roundings of 1.1e-16 relative to the sum of magnitudes."""
    for k, (n, G, ns) in enumerate(((1, 32, 0), (2047, 64, 1), (2049, 96, 3), (8192, 256, 8), (8193, 256, 1024),
                                    (8192 * 3 - 2048, 1024, 1025), (63 * 32 * 9, 96, 2049), (200001, 224, 5))):
        x = syn.draw_numpy(syn.NORMAL, n, 900 + k)
        x = syn.f32_to_bf16_bits(x) if dtype == "bf16" else x
        p, mn, sc, fp = gact.gact_compress_footprint(dev(x), G, 4, 5 + k, ns)
        p_ref, mn_ref, sc_ref = oracle.compress(x, G, 4, 5 + k)
        want, got = oracle.footprint(x, ns), fp.cpu().numpy()
        mag = float(np.abs(syn.bf16_bits_to_f32(x) if dtype == "bf16" else x).astype(np.float64).sum())
        assert abs(got[0] - want[0]) <= 60 * 1.2e-16 * mag, n
        assert np.array_equal(got[1:], want[1:]), n
        assert np.array_equal(p.cpu().numpy(), p_ref) and np.array_equal(mn.cpu().numpy(), mn_ref), n
        assert np.array_equal(sc.cpu().numpy(), sc_ref), n


@pytest.mark.parametrize("dtype,G,blocks", [("f32", 256, 8192 + 37), ("bf16", 96, 16384 + 300), ("bf16", 128, 32768 + 5)])
def test_fused_footprint_of_long_launches(gact, dtype, G, blocks):
    """Runs of 16 blocks and more per XCD with a last partial window, where a block's sum goes to the block's place;
    more sums than one addition takes.  Whole numbers, whose sum is exact in binary64."""
    bits, period = 2, 256
    n = blocks * 4 * (64 // (G // 32) * G) - 1234
    x = torch.arange(period, device="cuda", dtype=torch.float32).repeat(n // period + 1)[:n]
    x = x.to(torch.bfloat16) if dtype == "bf16" else x
    x[5] = 300.0                                       # no period over the whole of it
    full, rest = divmod(n, period)
    p, mn, sc, fp = gact.gact_compress_footprint(x, G, bits, 9, 7)
    got = fp.cpu().numpy()
    assert got[0] == full * (period * (period - 1) // 2) + rest * (rest - 1) // 2 + 295
    assert np.array_equal(got[1:], [float((j * n // 7) % period) for j in range(7)])
    assert all(torch.equal(a, b) for a, b in zip((p, mn, sc), gact.gact_compress(x, G, bits, 9)))


def test_footprint_of_more_blocks_than_one_addition_takes(gact):
    n = 32769 * 4096 + 5
    x = torch.arange(1024, device="cuda", dtype=torch.float32).repeat(n // 1024 + 1)[:n]
    full, rest = divmod(n, 1024)
    got = gact.gact_footprint(x, 7).cpu().numpy()
    assert got[0] == full * (1023 * 512) + rest * (rest - 1) // 2            # integers: exact in binary64
    assert np.array_equal(got[1:], [float((j * n // 7) % 1024) for j in range(7)])


@pytest.mark.parametrize("K", (103, 104, 105, 120))
def test_tables_in_the_arguments_and_in_the_workspace(gact, K):
    """The largest buffer list that travels in the kernel arguments, the smallest that is uploaded, and a
    longer list of which enough are empty; both types in one list."""
    sizes = [1 + (k * 977) % 9000 for k in range(K)]
    if K == 120:
        sizes[3:40:2] = [0] * len(sizes[3:40:2])
    half = K // 2
    g0 = buffers(sizes[:half], 10, "f32") + buffers(sizes[half:], 10, "bf16")
    g1 = buffers(sizes[:half], 500, "f32") + buffers(sizes[half:], 500, "bf16")
    got = gact.gact_sensitivity([dev(x) for x in g0], [dev(x) for x in g1], 2).item()
    assert got == pytest.approx(oracle.sensitivity(g0, g1, 2), rel=REL)
    means = [syn.draw_numpy(syn.NORMAL, n, 70 + k) if n else np.empty(0, np.float32) for k, n in enumerate(sizes)]
    d_means = [dev(m) for m in means]
    out = gact.gact_grad_stats_update([dev(x) for x in g0], d_means, 3).cpu().numpy()
    want = np.zeros(2)
    for g, m, d in zip(g0, means, d_means):
        if g.size:
            want += oracle.grad_stats_update(g, m, 3)
            assert np.array_equal(d.cpu().numpy().view(np.uint32), m.view(np.uint32))
    assert out == pytest.approx(want, rel=REL)


def test_calls_without_a_stream_go_to_the_current_one(gact):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert gact._stream(None) == s.cuda_stream
    assert gact._stream(None) == torch.cuda.current_stream().cuda_stream
    assert gact._stream(s) == s.cuda_stream and gact._stream(7) == 7


@pytest.mark.parametrize("sizes,dtypes", [((40000,), ("bf16",)), ((8192, 1, 50001, 4096, 4097), ("bf16", "f32", "bf16", "f32", "bf16")),
                                          (tuple(range(1, 40000, 300)), ("bf16",))])
def test_statistics_in_the_least_workspace(gact, sizes, dtypes):
    """A result pair for every 4,096 fp32 or 8,192 bf16 elements of a buffer, begun ones too, behind the table of 36
    bytes a buffer: enough although it is less than gact_reduce_workspace_bytes, and nothing behind it is
    touched; 16 bytes less is refused."""
    K = len(sizes)
    kinds = [dtypes[k % len(dtypes)] for k in range(K)]
    pairs = sum(-(-n // (4096 if d == "f32" else 8192)) for n, d in zip(sizes, kinds))
    need = (36 * K + 4 + 15) // 16 * 16 + 16 * pairs
    assert need < gact.gact_reduce_workspace_bytes(K, sum(sizes))
    g = [buffers([n], 20 + k, d)[0] for k, (n, d) in enumerate(zip(sizes, kinds))]
    means = [syn.draw_numpy(syn.NORMAL, n, 90 + k) for k, n in enumerate(sizes)]
    d_g, d_means = [dev(x) for x in g], [dev(m) for m in means]
    area = torch.full((need + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    with pytest.raises(gact.GactError):
        gact.gact_grad_stats_update(d_g, d_means, 3, workspace=area[:need - 16])
    out = gact.gact_grad_stats_update(d_g, d_means, 3, workspace=area[:need]).cpu().numpy()
    want = np.zeros(2)
    for x, m, d in zip(g, means, d_means):
        want += oracle.grad_stats_update(x, m, 3)
        assert np.array_equal(d.cpu().numpy().view(np.uint32), m.view(np.uint32))
    assert out == pytest.approx(want, rel=REL)
    assert (area[need:].cpu().numpy() == 0xA5).all()


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("blocks", (1, 63, 64, 65, 129, 255, 256, 257, 700, 4095, 4096, 4097 + 256))
def test_every_block_is_taken_once_in_any_order(gact, dtype, blocks):
    """Launches of no, one and several whole windows of eight runs (64 blocks of a sensitivity, 256 of a statistics
    step, which has them from 4,096 blocks on), with and without blocks behind them, in one buffer and in three.  Small whole numbers, a sum of which
    is exact; every chunk of a buffer has a value of its own, so that none can stand for another."""
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    for lists in (1, 3):
        per, total = (4096 if dtype == "f32" else 8192), 0
        g0, g1 = [], []
        for k in range(lists):
            n = max(blocks // lists, 1) * per - (3 if k else 0)
            i = torch.arange(n, device="cuda") // 2048 + 7 * k
            g0.append((i % 31).to(dt))
            g1.append((i % 31 - i % 13 - 1).to(dt))
            total += int(((i % 13 + 1) ** 2).sum())
        assert gact.gact_sensitivity(g0, g1, 1).item() == 0.5 * total
        means = [torch.zeros(g.numel(), device="cuda") for g in g0]
        out = gact.gact_grad_stats_update(g0, means, 1).cpu().tolist()
        want = float(sum((g.double() ** 2).sum() for g in g0))
        assert out == [want, want] and all(torch.equal(m, g.float()) for m, g in zip(means, g0))


@pytest.mark.parametrize("blocks", (1, 2, 511, 512, 513, 4096, 4097, 8193, 36865))
def test_sums_added_by_the_launch_itself_and_by_one_behind_it(gact, blocks):
    """Around the ends of rows of 512 results, of one adding block's eight rows, and of the 64 rows that a wavefront
    takes in one round.  The workspace holds room for two words a result (the launch adds them itself) or for one
    (a launch behind it does): the same order, so the same bits, whatever the workspace holds, and nothing behind
    that room is touched (in the calls after the first it holds what the ones before have left)."""
    n = blocks * 8192 - 5
    g0 = torch.randn(n, device="cuda", generator=torch.Generator("cuda").manual_seed(blocks)).to(torch.bfloat16)
    g1 = g0 * 0.5
    want = 0.5 * 9.0 * sum(float(((a.double() - b.double()) ** 2).sum()) for a, b in zip(g0.split(1 << 26), g1.split(1 << 26)))
    table = (36 + 4 + 15) // 16 * 16
    both = torch.full((table + 16 * blocks + 64,), 0xFF, dtype=torch.uint8, device="cuda")
    got = []
    for nbytes in (16, 16, 8, 16):
        if len(got) == 3:
            both.zero_()
        before = both.clone()
        out = torch.zeros(1, dtype=torch.float64, device="cuda")
        gact.gact_sensitivity([g0], [g1], 2, out=out, workspace=both[:table + nbytes * blocks])
        got.append(out.item())
        assert torch.equal(both[table + nbytes * blocks:], before[table + nbytes * blocks:]), (len(got), nbytes)
    assert got == [got[0]] * 4
    assert got[0] == pytest.approx(want, rel=1e-12)
    with pytest.raises(gact.GactError):
        gact.gact_sensitivity([g0], [g1], 2, workspace=both[:table + 8 * blocks - 1])


def test_sensitivities_of_two_streams_at_a_time(gact):
    """Each call adds its own results in its own workspace, also while another runs."""
    gen = torch.Generator("cuda").manual_seed(3)
    pairs = [[torch.randint(0, 4, (5_000_000 + 4096 * k,), device="cuda", generator=gen).float() for _ in range(2)] for k in range(4)]
    want = [0.5 * float(((a - b).double() ** 2).sum()) for a, b in pairs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in pairs]
    spaces = [torch.empty(gact.gact_reduce_workspace_bytes(1, a.numel()), dtype=torch.uint8, device="cuda") for a, _ in pairs]
    results = torch.zeros(len(pairs), 10, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    for r in range(10):
        for k, (a, b) in enumerate(pairs):
            gact.gact_sensitivity([a], [b], 1, out=results[k, r:r + 1], workspace=spaces[k], stream=streams[k])
    torch.cuda.synchronize()
    assert results.cpu().tolist() == [[w] * 10 for w in want]


@pytest.mark.parametrize("K", (1, 105))
@pytest.mark.parametrize("blocks,shift", [(8191, 0), (8192, 0), (8192, 4), (8193 + 40, 0)])
def test_statistics_in_wide_blocks(gact, K, blocks, shift):
    """The shortest launch of wide blocks and the longest of the others, means that start on a line and 16 bytes
    behind one, buffers that end inside a chunk, inside a piece and on a chunk's end; the tables of both kinds.
    Element by element as torch computes the three operations; sums of whole numbers, exact in binary64."""
    sizes = [4096 * (blocks - K + 1)] + [4096] * (K - 1)
    if blocks % 2:
        sizes[0] -= 4093
        sizes[-1] -= 1 if K > 1 else 0
    g, means = [], []
    for k, n in enumerate(sizes):
        g.append(((torch.arange(n, device="cuda") * 7 + k) % 33 - 16).float())
        room = torch.full((n + shift + 32,), 5.0, device="cuda")
        room[shift:shift + n] = ((torch.arange(n, device="cuda") + 3 * k) % 17 - 8).float()
        means.append(room)
    views = [m[shift:shift + n] for m, n in zip(means, sizes)]
    want = [v + (x - v) * 0.5 for x, v in zip(g, views)]
    out = gact.gact_grad_stats_update(g, views, 2).cpu().tolist()
    assert out == [float(sum((x.double() ** 2).sum() for x in g)), float(sum((w.double() ** 2).sum() for w in want))]
    for m, w in zip(means, want):
        assert torch.equal(m[shift:shift + w.numel()], w)
        assert bool((m[:shift] == 5.0).all()) and bool((m[shift + w.numel():] == 5.0).all())


@pytest.mark.parametrize("n", (2048, 2049, 8192 * 512, 8192 * 2049 + 7))
def test_footprints_recorded_into_a_graph(gact, n):
    """A recorded call adds its sums in a launch behind, whose replays share one tag; sizes of one tile (no room for
    two words a sum), of one row of sums and of more rows than one adding block has.  Replayed on changed inputs
    with eager calls on the same workspace in between, and compared with an eager call's bits."""
    G, bits, ns = 256, 2, 5
    x = torch.empty(n, device="cuda")
    p, mn, sc = gact.alloc_compressed(n, G, bits, x.device)
    ws = torch.zeros(gact.gact_compress_footprint_workspace_bytes(n, G), dtype=torch.uint8, device="cuda")
    fp = torch.zeros(1 + ns, dtype=torch.float64, device="cuda")
    gen = torch.Generator("cuda").manual_seed(n)
    x.normal_(generator=gen)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        gact.gact_compress_footprint(x, G, bits, 3, ns, p, mn, sc, fp, ws)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gact.gact_compress_footprint(x, G, bits, 3, ns, p, mn, sc, fp, ws)
    for _ in range(4):
        x.normal_(generator=gen)
        graph.replay()
        got = [t.clone() for t in (p, mn, sc, fp)]
        fp.zero_()
        gact.gact_compress_footprint(x, G, bits, 3, ns, p, mn, sc, fp, ws)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, (p, mn, sc, fp)))
        assert fp[0].item() == pytest.approx(float(x.double().sum()), abs=60 * 1.2e-16 * float(x.abs().double().sum()))
