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
