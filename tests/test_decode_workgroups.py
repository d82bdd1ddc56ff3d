"""The number of workgroups of a decode call and the workspace that follows from it: a workspace for more chunks serves
fewer, and what fitted the fixed array of moqae_decode_attn_static still does; short calls on many workgroups against the
oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


def test_workspace_grows_with_chunks_and_keeps_the_static_limit():
    from paper_2506_07533_amd import binding as mq
    limit = mq.static_scratch_bytes()
    rng = np.random.default_rng(3)
    cus = 256
    for _ in range(4000):
        rep = int(rng.choice([1, 1, 2, 4, 8])); G = 64 if rep == 8 else int(rng.choice([32, 64]))
        H = int(rng.choice([1, 2, 5, 8, 32, 40, 64, 100, 513])); B = int(rng.choice([1, 2, 3, 8, 40, 100])); N = int(rng.choice([8, 32, 64, 128, 256]))
        if B * H > 65535:
            continue
        cfg = mq.Cfg(B, H * rep, H, 128, N, G)
        C = int(rng.choice([0, 1, 2, 5, 17, 100, 1024, 3000]))
        sizes = [mq.decode_workspace_bytes(cfg, c) for c in (C, C + 1, C + 70, C + 4000)]
        assert sizes == sorted(sizes), (B, H, rep, N, C)
        ragged = [mq.decode_workspace_bytes_ragged(cfg, c) for c in (C, C + 1, C + 70, C + 4000)]
        assert ragged == sorted(ragged), (B, H, rep, N, C)
        assert all(r >= s for r, s in zip(ragged, sizes)), (B, H, rep, N, C)   # a ragged workspace serves uniform calls
        if torch.cuda.is_available():
            cus = torch.cuda.get_device_properties(0).multi_processor_count
        # one wavefront per ticket of 128 tokens: the size of a workspace by the rule for long caches alone
        BH, NW = B * H, 0
        NW = max(1, min(cus, (BH * (C * (N // 128 if N >= 256 else 1) + (N - 1 + 127) // 128) + 7) // 8))
        slots = min(NW, 8 * NW // (BH + 7) + 3 if BH <= 1024 else NW // BH + 2)
        segment = min(1024, 8192 // max(N // 16, 1))
        plain = (BH * max(1, -(-C // segment)) * 256 + 8 * BH + 255) // 256 * 256 + B * H * rep * slots * 130 * 4
        assert sizes[0] >= plain
        assert plain > limit or sizes[0] <= limit, (B, H, rep, N, C, plain, sizes[0])


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,N,G,C,T", [
    (1, 1, 1, 128, 64, 60, 100),     # 32 workgroups on one row
    (1, 3, 3, 64, 32, 1, 63),        # fewer units than wavefronts
    (2, 8, 8, 256, 64, 1, 200),      # more workgroups than units in a row's batches
    (1, 8, 2, 128, 64, 3, 127),      # grouped queries
    (1, 40, 40, 128, 64, 0, 90),     # residual only
    (70, 8, 8, 64, 64, 1, 30),       # more rows than workgroups
    (41, 25, 25, 64, 64, 9, 30),     # more than 1024 rows, whose costs are not weighed, most of them cut
    (130, 8, 8, 32, 64, 5, 3),
    (205, 10, 5, 128, 64, 2, 17),    # the same with grouped queries
    (1, 40, 40, 64, 64, 30, 7),      # 240 workgroups, six a row
    (3, 40, 40, 64, 64, 6, 40),      # 256 workgroups on 120 rows: rows are cut
    (1, 5, 5, 8, 64, 40, 3), (1, 32, 32, 32, 64, 15, 20),   # short chunks, a multiple of the rows
])
def test_short_calls(ref, B, Hq, Hkv, N, G, C, T):
    """24-bit fixed point and binary32 sums: 2e-5 of a row's largest output; grouped queries hold their weights in fp16 (2e-3)."""
    import test_gpu_parity as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_07533_amd import binding as mq
    assert P._attn_case(mq, ref, B, Hq, Hkv, N, G, C, T, (2, 4, 8, 16), 7 * C + T) <= (2e-5 if Hq == Hkv else P.ATTN_TOL)


@pytest.mark.gpu
@pytest.mark.parametrize("H,N,C", [(8, 64, 8), (4, 32, 3), (1, 128, 30)])
def test_ragged_call_needs_its_own_workspace_only(ref, H, N, C):
    """Short caches: a uniform call takes more workgroups, and its workspace is the larger one.  A ragged call runs on what its
    own rule gives (a ticket of 128 tokens per wavefront, a partial per workgroup and row) and is refused below it."""
    import test_gpu_parity as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_07533_amd import binding as mq
    rng = np.random.default_rng(N)
    cfg, rcfg = P._cfgs(mq, ref, 2, H, H, N, 64, (2, 4, 8, 16), 0)
    cus, rows = torch.cuda.get_device_properties(0).multi_processor_count, 2 * H
    n_wg = max(1, min(cus, (rows * (C + (N - 1 + 127) // 128) + 7) // 8))
    own = (rows * 256 + 8 * rows + 255) // 256 * 256 + rows * n_wg * 130 * 4
    assert own < mq.decode_workspace_bytes_ragged(cfg, C)
    K, V = P._rand_kv(rng, 2, H, C * N)
    expert = rng.integers(0, 4, (rows, C)).astype(np.uint8)
    (arena, used, off, status), (arena_ref, used_ref, off_ref, _) = P._pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert)
    q = rng.standard_normal((2, H, 128), dtype=np.float32).astype(np.float16)
    Kt = torch.zeros((2, H, N, 128), dtype=torch.float16, device="cuda")
    counts, tails = (torch.tensor(x, dtype=torch.int32, device="cuda") for x in ([C, 1], [0, 0]))
    out = torch.full((2, H, 128), float("nan"), dtype=torch.float32, device="cuda")
    room = torch.full((own + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    call = lambda ws: mq.decode_attn_ragged(cfg, P._dev(q), arena, off, P._dev(expert), counts, C, Kt, Kt, tails, 128 ** -0.5, out, ws)
    with pytest.raises(mq.MoqaeError) as e:
        call(room[:own - 256])
    assert e.value.code == mq.E_WORKSPACE
    call(room[:own])
    torch.cuda.synchronize()
    assert bool((room[own:] == 0xA5).all())                              # nothing beyond it is written
    whole = ref.decode_attn(rcfg, q, arena_ref, off_ref, expert, C, None, None, 0, 128 ** -0.5)
    first = ref.decode_attn(rcfg, q, arena_ref, off_ref, expert, 1, None, None, 0, 128 ** -0.5)
    want = np.stack([whole[0], first[1]])
    assert (np.abs(out.cpu().numpy() - want).max(-1) / np.abs(want).max(-1)).max() <= 2e-5


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,N,G,C,heavy", [
    (1, 8, 8, 64, 32, 33, False),        # an even share of the tickets for each of a row's workgroups
    (1, 8, 2, 128, 64, 1, False),        # more workgroups than tickets
    (240, 1, 1, 64, 64, 3, False),       # one workgroup per row, which writes the output
    (60, 16, 4, 32, 64, 5, False),       # the same for grouped queries
    (350, 2, 2, 64, 64, 2, False),       # more rows than compute units
    (4, 16, 16, 64, 64, 80, False),      # costs added up by the workgroups, table rows of whole 16-byte pieces
    (4, 16, 16, 64, 64, 70, False),      # table rows that begin anywhere
    (4, 16, 16, 64, 64, 70, True),       # one row costs several times the others: intervals
    (2, 64, 32, 64, 64, 65, True),
    (8, 32, 32, 32, 64, 70, False),      # costs in the workspace, one workgroup per row
    (8, 32, 32, 32, 64, 70, True),
    (8, 16, 16, 32, 64, 150, False),     # costs in the workspace, two workgroups per row share its tickets by the counter
    (8, 16, 16, 32, 64, 150, True),      # ... one row costs several times the others: intervals by the same costs
    (4, 64, 32, 64, 64, 150, False),     # the same for grouped queries
    (4, 64, 32, 64, 64, 150, True),
    (1, 8, 8, 16, 64, 70, False),        # short chunks: every P-th unit for each of a row's workgroups
    (1, 1, 1, 8, 64, 1100, False),       # ... in two segments
    (2, 8, 2, 8, 64, 1100, False),       # two segments of a row
])
def test_fixed_workgroups_per_row(ref, B, Hq, Hkv, N, G, C, heavy):
    """Calls on a plan, whose residual grows, and without one, on both sides of every line of the rule; tolerances as in test_short_calls."""
    import test_gpu_parity as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_07533_amd import binding as mq
    rng = np.random.default_rng(B * C + N)
    cfg, rcfg = P._cfgs(mq, ref, B, Hq, Hkv, N, G, (2, 4, 8, 16), 1)
    K, V = P._rand_kv(rng, B, Hkv, C * N + N)
    BH = B * Hkv
    expert = np.tile(rng.integers(0, 4, (1, C)).astype(np.uint8), (BH, 1))   # rows of equal cost
    if heavy:
        expert[:] = 0
        expert[BH // 3] = 3
    (arena, used, off, status), (arena_ref, used_ref, off_ref, _) = P._pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert)
    ed, scale = P._dev(expert), 128 ** -0.5
    ws = torch.full((mq.decode_workspace_bytes(cfg, C),), 0xFF, dtype=torch.uint8, device="cuda")
    mq.decode_plan(cfg, ed, C, ws)
    for rows, planned in ((1, True), (N - 1, True), (0, True), (N // 2, False)):   # a planned call leaves the counters as it found them
        q = rng.standard_normal((B, Hq, 128), dtype=np.float32).astype(np.float16)
        Kt = np.full((B, Hkv, N, 128), np.nan, np.float16); Vt = Kt.copy()
        Kt[:, :, :rows] = K[:, :, C * N:C * N + rows]; Vt[:, :, :rows] = V[:, :, C * N:C * N + rows]
        want = ref.decode_attn(rcfg, q, arena_ref, off_ref, expert, C, Kt, Vt, rows, scale)
        out = torch.full((B, Hq, 128), float("nan"), dtype=torch.float32, device="cuda")
        mq.decode_attn(cfg, P._dev(q), arena, off, ed, C, P._dev(Kt), P._dev(Vt), rows, scale, out, ws, planned=planned)
        torch.cuda.synchronize()
        err = (np.abs(out.cpu().numpy() - want).max(-1) / np.abs(want).max(-1)).max()
        assert err <= (2e-5 if Hq == Hkv else P.ATTN_TOL), (rows, planned, err)
