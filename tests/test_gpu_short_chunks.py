"""Chunks shorter than a window of 64 tokens share wavefronts in the routing kernel, take a wavefront per side and 32 tokens in the
packing kernel and share units in the decode kernel: windows that end inside a row, frozen chunks inside a window, calls that begin
inside one, odd numbers of chunk sides (bit-exact against the CPU oracle); units with fewer chunks than they hold."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import test_gpu_parity as T                                              # noqa: E402  (helpers only)

mq = T.mq


@pytest.mark.parametrize("B,Hkv,N,C,M,freeze,c0,pad", [
    (1, 3, 32, 7, 4, 1, 0, 0),          # a window of one chunk at the end of every row
    (2, 2, 32, 9, 8, 3, 1, 8),          # the call begins in the middle of a window; rows 136 elements apart
    (1, 2, 16, 5, 3, 2, 0, 0),
    (1, 5, 8, 19, 2, 10, 3, 0),         # a window frozen as a whole, one in part
    (3, 1, 8, 1, 1, 0, 0, 0),
    (2, 40, 32, 210, 4, 1, 0, 0),       # more windows than wavefronts of the grid: several each
    (2, 3, 32, 9, 4, 9, 0, 0),          # every chunk of the call frozen: no windows
    (1, 40, 8, 150, 4, 149, 2, 0),      # one chunk left; more frozen chunks than lanes
    (3, 30, 16, 70, 8, 65, 1, 8),
    (1, 1, 32, 1, 4, 5, 0, 0),
])
def test_route_windows_of_short_chunks(mq, ref, B, Hkv, N, C, M, freeze, c0, pad):
    rng = np.random.default_rng(N * 1000 + C)
    bits = (16, 2, 4, 8, 2, 4, 8, 16)[:M]
    cfg, rcfg = T._cfgs(mq, ref, B, Hkv, Hkv, N, 32, bits, freeze)
    K, _ = T._rand_kv(rng, B, Hkv, C * N)
    W = [(rng.standard_normal(s) * 0.3).astype(np.float16) for s in ((128, M), (128, M), (M, M))]
    e_ref, v_ref = ref.route_chunks(rcfg, K, 0, C, *W)
    Kd = torch.full((B, Hkv, C * N, 128 + pad), float("nan"), dtype=torch.float16, device="cuda")
    Kd[..., :128] = T._dev(K)
    expert = torch.full((B * Hkv, C), 255, dtype=torch.uint8, device="cuda")
    votes = torch.full((B * Hkv, C, M), -1, dtype=torch.int32, device="cuda")
    mq.route_chunks(cfg, Kd[..., :128], c0, C, *[T._dev(w) for w in W], None, expert, votes)
    torch.cuda.synchronize()
    e, v = expert.cpu().numpy(), votes.cpu().numpy()
    assert np.array_equal(e[:, c0:], e_ref[:, c0:]) and np.array_equal(v[:, c0:], v_ref[:, c0:])
    assert (e[:, :c0] == 255).all() and (v[:, :c0] == -1).all()         # entries before the call's chunks are not touched


@pytest.mark.parametrize("B,Hkv,N,G,C,kpc", [
    (1, 2, 8, 64, 5, 0), (2, 1, 16, 32, 3, 0), (1, 3, 32, 32, 7, 1), (1, 3, 32, 64, 1, 0), (2, 2, 64, 64, 5, 1), (1, 1, 8, 32, 1, 0),
])
def test_pack_wavefront_per_side(mq, ref, B, Hkv, N, G, C, kpc):
    rng = np.random.default_rng(N * 100 + G + C)
    cfg, rcfg = T._cfgs(mq, ref, B, Hkv, Hkv, N, G, (2, 4, 8, 16), 0, kpc)
    K, V = T._rand_kv(rng, B, Hkv, C * N)
    expert = rng.integers(0, 4, (B * Hkv, C)).astype(np.uint8)
    (arena, used, off, status), (arena_ref, used_ref, off_ref, st_ref) = T._pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert)
    assert int(status.item()) == st_ref == 0 and int(used.item()) == int(used_ref[0])
    assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    assert np.array_equal(arena.cpu().numpy(), arena_ref)


@pytest.mark.parametrize("B,Hkv,N,G,C,kpc,bits", [
    (1, 2, 8, 64, 1, 0, (2, 4, 8, 16)), (1, 3, 8, 32, 6, 0, (2, 4, 8, 16)), (2, 2, 8, 64, 11, 0, (8,)),      # groups of four chunks, the last in part
    (1, 2, 16, 32, 1, 0, (2, 4, 8, 16)), (1, 3, 16, 64, 5, 0, (2, 4, 8, 16)), (1, 2, 16, 64, 4, 0, (4,)),    # pairs
    (1, 3, 8, 64, 13, 0, (16,)), (1, 2, 16, 32, 3, 0, (16,)), (1, 3, 8, 32, 61, 0, (16, 16, 16, 2)),         # groups of raw chunks alone
    (1, 2, 32, 32, 3, 0, (8,)), (1, 2, 32, 32, 5, 1, (2, 4, 8, 16)),
    (1, 2, 64, 64, 3, 1, (2, 4, 8, 16)), (1, 2, 64, 32, 3, 1, (8,)), (2, 1, 128, 64, 5, 1, (2, 4, 8, 16)),   # a group of 64 by two wavefronts
    (1, 2, 192, 64, 3, 0, (8,)), (1, 3, 192, 32, 4, 1, (2, 4, 8, 16)), (1, 2, 256, 32, 4, 0, (2, 4, 8, 16)), # three and four parts of a chunk
])
def test_pack_rows_by_lines(mq, ref, B, Hkv, N, G, C, kpc, bits):
    """K and V as views of a [B, S, 3, H, D] tensor (rows far apart), the chunks after the first two, an arena that ends where
    the last block does and bytes behind it that stay: byte for byte the oracle's."""
    rng = np.random.default_rng(N * 1000 + G + C + kpc)
    M, BH, C0 = len(bits), B * Hkv, 2
    cfg, rcfg = T._cfgs(mq, ref, B, Hkv, Hkv, N, G, bits, 0, kpc)
    K, V = T._rand_kv(rng, B, Hkv, (C0 + C) * N)
    qkv = torch.zeros(B, (C0 + C) * N, 3, Hkv, 128, dtype=torch.float16, device="cuda")
    qkv[:, :, 1], qkv[:, :, 2] = T._dev(K).transpose(1, 2), T._dev(V).transpose(1, 2)
    Kd, Vd = qkv[:, :, 1].transpose(1, 2), qkv[:, :, 2].transpose(1, 2)
    expert = rng.integers(0, M, (BH, C0 + C)).astype(np.uint8)
    need = sum((ref.chunk_block_bytes(rcfg, bits[e]) + 255) // 256 * 256 for e in expert[:, C0:].ravel())
    guard = 4096
    arena_ref = np.zeros(need, np.uint8); used_ref = np.zeros(1, np.uint64); off_ref = np.zeros((BH, C0 + C), np.uint64)
    assert ref.quantize_pack(rcfg, K, V, C0, C0 + C, expert, arena_ref, used_ref, off_ref) == 0
    arena = torch.full((need + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    arena[:need] = 0
    used = torch.zeros(1, dtype=torch.int64, device="cuda"); status = torch.zeros(1, dtype=torch.int32, device="cuda")
    off = torch.zeros((BH, C0 + C), dtype=torch.int64, device="cuda")
    mq.quantize_pack(cfg, Kd, Vd, C0, C0 + C, T._dev(expert), arena[:need], used, off, status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and int(used.item()) == int(used_ref[0])
    assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    got = arena.cpu().numpy()
    assert np.array_equal(got[:need], arena_ref) and (got[need:] == 0xA5).all()


@pytest.mark.parametrize("N,G,kpc", [(8, 64, 0), (8, 32, 0), (16, 32, 0), (32, 32, 0), (32, 32, 1), (64, 64, 1), (64, 32, 1), (128, 32, 0)])
def test_pack_streaming_loads(mq, ref, N, G, kpc):
    """Calls on more than 384 MiB of K and V: the keys and values of 1000 heads are views of one head's."""
    BH, C, bits = 1000, 896 // N, (2, 4, 8, 16)
    assert BH * C * N * 512 > 384 << 20
    rng = np.random.default_rng(N + G + kpc)
    cfg, rcfg = T._cfgs(mq, ref, 1, BH, BH, N, G, bits, 0, kpc)
    K, V = T._rand_kv(rng, 1, 1, C * N)
    expert = rng.choice(4, (BH, C), p=(0.6, 0.3, 0.05, 0.05)).astype(np.uint8)
    sizes = np.array([(ref.chunk_block_bytes(rcfg, b) + 255) // 256 * 256 for b in bits])[expert].ravel()
    want = (np.cumsum(sizes) - sizes).reshape(BH, C)
    arena = torch.zeros(int(sizes.sum()), dtype=torch.uint8, device="cuda")
    used = torch.zeros(1, dtype=torch.int64, device="cuda"); status = torch.zeros(1, dtype=torch.int32, device="cuda")
    off = torch.zeros((BH, C), dtype=torch.int64, device="cuda")
    mq.quantize_pack(cfg, T._dev(K).expand(1, BH, -1, -1), T._dev(V).expand(1, BH, -1, -1), 0, C, T._dev(expert), arena, used, off, status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and int(used.item()) == arena.numel() and np.array_equal(off.cpu().numpy(), want)
    got, blocks = arena.cpu().numpy(), {}
    rows = np.concatenate([[0, BH - 1], rng.choice(BH, min(BH, 4000 // C), replace=False)])
    for u in rows:
        for c in range(C):
            b = bits[expert[u, c]]
            if (b, c) not in blocks:
                blocks[b, c] = ref.pack_chunk(rcfg, b, K[0, 0, c * N:(c + 1) * N], V[0, 0, c * N:(c + 1) * N])
            blk = blocks[b, c]
            assert np.array_equal(got[want[u, c]:want[u, c] + blk.size], blk), (u, c, b)


@pytest.mark.parametrize("N", [8, 64])
def test_refused_call_reads_no_rows(mq, N):
    """A call on a status that is set is a no-op in time too: on 537 MB of K and V about 20 us, a sixth of an accepted call, and
    two thirds of one if it read them."""
    BH, C = 32, (1 << 20) // (32 * N)
    cfg = mq.Cfg(1, BH, BH, 128, N, 64, (2, 4, 8, 16), 0)
    K, V = (torch.zeros(1, BH, C * N, 128, dtype=torch.float16, device="cuda") for _ in range(2))
    expert = torch.ones(BH, C, dtype=torch.uint8, device="cuda")
    arena = torch.zeros(mq.chunk_block_bytes(cfg, 4) * BH * C + 256 * BH * C, dtype=torch.uint8, device="cuda")
    used = torch.zeros(1, dtype=torch.int64, device="cuda"); off = torch.zeros(BH, C, dtype=torch.int64, device="cuda")
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def fastest(word):
        status = torch.full((1,), word, dtype=torch.int32, device="cuda")
        times = []
        for _ in range(5):
            begin.record()
            for _ in range(10):
                used.zero_()
                mq.quantize_pack(cfg, K, V, 0, C, expert, arena, used, off, status)
            end.record()
            torch.cuda.synchronize()
            times.append(begin.elapsed_time(end))
        assert int(status.item()) == word
        return min(times)

    fastest(0)
    assert fastest(mq.E_ARENA) < 0.4 * fastest(0)


SMALL, LARGE = (8, (2, 4, 8, 16, 16, 2)), (256, (2, 16, 8, 4, 16, 8))       # blocks of up to 16 and 512 units of 256 bytes


@pytest.mark.parametrize("BH,C,c0,blocks", [
    (1, 2049, 0, SMALL), (3, 1040, 16, SMALL), (130, 33, 0, SMALL), (300, 47, 32, SMALL), (1024, 3, 0, SMALL), (5, 1023, 0, SMALL),
    (1024, 67, 0, SMALL), (300, 231, 16, SMALL), (1000, 48, 0, SMALL),       # 5120, 4500 and 3000 pieces: a second batch, the second to fourth piece of the first
    (130, 33, 0, LARGE), (7, 147, 16, LARGE),                                # sizes of two bytes
])
def test_pack_plan_per_row(mq, ref, BH, C, c0, blocks):
    """Offsets, the arena's end and the verdict on an expert out of range, wherever it stands: more than a pass of 1024 chunks in a row,
    pieces of 16 decisions that are whole or end early, more than a batch of four pieces for each of the 1024 threads."""
    rng = np.random.default_rng(BH * 7 + C)
    N, bits = blocks
    cfg, rcfg = T._cfgs(mq, ref, 1, BH, BH, N, 64, bits, 0)
    cols = (c0 + C + 15) // 16 * 16
    size = np.array([(ref.chunk_block_bytes(rcfg, b) + 255) // 256 * 256 for b in bits])
    K = torch.zeros(1, 1, (c0 + C) * N, 128, dtype=torch.float16, device="cuda").expand(1, BH, -1, -1)
    expert = rng.integers(0, len(bits), (BH, cols)).astype(np.uint8)
    expert[:, :c0] = 200; expert[:, c0 + C:] = 200                           # not the call's
    sizes = size[expert[:, c0:c0 + C]]
    need = int(sizes.sum())
    want = 512 + (np.cumsum(sizes.ravel()) - sizes.ravel()).reshape(BH, C)
    arena = torch.zeros(512 + need, dtype=torch.uint8, device="cuda")
    off = torch.full((BH, cols), -7, dtype=torch.int64, device="cuda")
    used = torch.full((1,), 300, dtype=torch.int64, device="cuda"); status = torch.zeros(1, dtype=torch.int32, device="cuda")
    mq.quantize_pack(cfg, K, K, c0, c0 + C, T._dev(expert), arena, used, off, status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and int(used.item()) == 512 + need
    o = off.cpu().numpy()
    assert np.array_equal(o[:, c0:c0 + C], want) and (o[:, :c0] == -7).all() and (o[:, c0 + C:] == -7).all()
    for u, c, e in [(0, c0, 6), (BH - 1, c0 + C - 1, 255), (BH // 2, c0 + C // 2, 129), (BH - 1, c0 + C - 1, 7), (BH - 1, c0, 6)]:
        bad = expert.copy(); bad[u, c] = e
        used.fill_(300); off.fill_(-7); status.zero_()
        mq.quantize_pack(cfg, K, K, c0, c0 + C, T._dev(bad), arena, used, off, status)
        torch.cuda.synchronize()
        assert int(status.item()) == mq.E_INVAL and int(used.item()) == 300 and (off == -7).all().item()


@pytest.mark.parametrize("B,Hkv,N,G,C,tail,mix", [
    (1, 2, 32, 64, 9, 31, (1, 0, 0, 0)),        # 2 bits: four chunks a unit, the last unit holds one
    (2, 1, 32, 32, 7, 5, (0, 1, 0, 0)),         # 4 bits: two a unit
    (1, 3, 16, 64, 13, 0, (0.4, 0.3, 0.2, 0.1)),
    (1, 1, 16, 32, 11, 15, (0, 0, 1, 0)),       # 8 bits: two a unit
    (1, 2, 8, 64, 17, 7, (1, 0, 0, 0)),         # half slices: eight chunks a unit, every second run of 8 tokens masked
    (1, 2, 8, 32, 21, 3, (0, 0.5, 0.5, 0)),     # eight and four a unit
    (1, 1, 8, 64, 1, 0, (1, 0, 0, 0)),
    (1, 2, 32, 64, 5, 17, (0, 0, 0, 1)),        # raw rows: two units a chunk
    (1, 1, 8, 32, 1100, 1, (0.6, 0.3, 0.05, 0.05)),   # more chunks than a row segment holds
    (1, 2, 32, 32, 1030, 0, (0.3, 0.3, 0.2, 0.2)),
    (2, 2, 32, 64, 0, 9, (1, 0, 0, 0)),         # residual only
])
def test_units_of_several_chunks(mq, ref, B, Hkv, N, G, C, tail, mix):
    """24-bit fixed point (2^-24 of the largest query entry / of a unit's largest weight) and binary32 sums over at most
    33 k tokens: below 2e-5 of a row's largest output; a chunk that is misplaced or counted twice shows as 1e-3 and more."""
    rng = np.random.default_rng(N * 10000 + C)
    expert = rng.choice(4, size=(B * Hkv, max(C, 1)), p=mix).astype(np.uint8)
    assert T._attn_case(mq, ref, B, Hkv, Hkv, N, G, C, tail, (2, 4, 8, 16), C + N, expert=expert) <= 2e-5


@pytest.mark.parametrize("B,Hkv,N,G,C,mix,kpc", [
    (2, 2, 32, 64, 37, (0.3, 0.3, 0.2, 0.2), 0),      # units of one chunk (8 bits, raw) beside units of several
    (1, 3, 16, 32, 50, (0.4, 0.2, 0.2, 0.2), 0),
    (1, 2, 8, 64, 1100, (0.4, 0.3, 0.2, 0.1), 0),     # two segments
    (2, 1, 32, 32, 45, (0.3, 0.3, 0.2, 0.2), 1),      # keys per channel
    (1, 2, 32, 32, 1030, (0.25, 0.25, 0.25, 0.25), 1),
    (1, 1, 32, 32, 9, (0, 0, 1, 0), 1),
    (1, 2, 8, 32, 70, (0, 0, 0, 1), 0),
])
def test_units_of_several_chunks_on_a_plan(mq, ref, B, Hkv, N, G, C, mix, kpc):
    """Row costs of a plan (made without the residual's length), then calls with a growing residual; tolerance as above."""
    rng = np.random.default_rng(N * 10 + C)
    cfg, rcfg = T._cfgs(mq, ref, B, Hkv, Hkv, N, G, (2, 4, 8, 16), 0, kpc)
    K, V = T._rand_kv(rng, B, Hkv, C * N + N)
    expert = rng.choice(4, size=(B * Hkv, C), p=mix).astype(np.uint8)
    (arena, used, off, status), (arena_ref, used_ref, off_ref, st_ref) = T._pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert)
    ws = torch.empty(mq.decode_workspace_bytes(cfg, C), dtype=torch.uint8, device="cuda").fill_(0xFF)
    out = torch.zeros((B, Hkv, 128), dtype=torch.float32, device="cuda")
    ed, scale = T._dev(expert), 128 ** -0.5
    mq.decode_plan(cfg, ed, C, ws)
    for rows in (0, 1, N // 2 + 1, N - 1):
        q = rng.standard_normal((B, Hkv, 128), dtype=np.float32).astype(np.float16)
        Kt = np.full((B, Hkv, N, 128), np.nan, np.float16); Vt = np.full_like(Kt, np.inf)   # rows past n_tail hold junk
        Kt[:, :, :rows] = K[:, :, C * N:C * N + rows]; Vt[:, :, :rows] = V[:, :, C * N:C * N + rows]
        want = ref.decode_attn(rcfg, q, arena_ref, off_ref, expert, C, Kt, Vt, rows, scale)
        out.fill_(float("nan"))
        mq.decode_attn(cfg, T._dev(q), arena, off, ed, C, T._dev(Kt), T._dev(Vt), rows, scale, out, ws, planned=True)
        torch.cuda.synchronize()
        err = (np.abs(out.cpu().numpy() - want).max(-1) / np.abs(want).max(-1)).max()
        assert err <= 2e-5, (rows, err)


@pytest.mark.parametrize("Hkv,N,C,M,freeze", [
    (2, 128, 3, 4, 1), (1, 96, 5, 3, 0), (3, 224, 2, 8, 0), (2, 256, 1, 2, 0),   # a wavefront per 64 tokens of a chunk
    (130, 96, 8, 4, 1), (64, 160, 13, 5, 0), (100, 224, 8, 8, 0),               # more than four (three) per compute unit: a wavefront per chunk
    (40, 128, 60, 1, 0), (40, 128, 60, 2, 55),                                  # one expert; two, and few chunks that are not frozen
])
def test_route_few_and_many_long_chunks(mq, ref, Hkv, N, C, M, freeze):
    assert T._persistent_chunks(M, N, Hkv * C) == (Hkv >= 40)
    rng = np.random.default_rng(N + C)
    cfg, rcfg = T._cfgs(mq, ref, 1, Hkv, Hkv, N, 32, (16, 2, 4, 8, 2, 4, 8, 16)[:M], freeze)
    K, _ = T._rand_kv(rng, 1, Hkv, C * N)
    W = [(rng.standard_normal(s) * 0.3).astype(np.float16) for s in ((128, M), (128, M), (M, M))]
    bias = (rng.standard_normal(M) * 0.05).astype(np.float32)
    e_ref, v_ref = ref.route_chunks(rcfg, K, 0, C, *W, bias)
    expert = torch.full((Hkv, C), 255, dtype=torch.uint8, device="cuda")
    votes = torch.full((Hkv, C, M), -1, dtype=torch.int32, device="cuda")
    mq.route_chunks(cfg, T._dev(K), 0, C, *[T._dev(w) for w in W], T._dev(bias), expert, votes)
    torch.cuda.synchronize()
    assert np.array_equal(expert.cpu().numpy(), e_ref) and np.array_equal(votes.cpu().numpy(), v_ref)


@pytest.mark.parametrize("BH,C", [(64, 16), (41, 25), (1, 1025), (64, 32)])    # 1024, 1025 and 2048 chunks: one workgroup plans, or one per row
def test_pack_plan_of_small_tables(mq, ref, BH, C):
    rng = np.random.default_rng(BH + C)
    cfg, rcfg = T._cfgs(mq, ref, 1, BH, BH, 8, 64, (2, 4, 8, 16), 0)
    K, V = T._rand_kv(rng, 1, BH, C * 8)
    expert = rng.integers(0, 4, (BH, C)).astype(np.uint8)
    (arena, used, off, status), (arena_ref, used_ref, off_ref, st_ref) = T._pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert, start=300)
    assert int(status.item()) == st_ref == 0 and int(used.item()) == int(used_ref[0])
    assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    assert np.array_equal(arena.cpu().numpy(), arena_ref)
