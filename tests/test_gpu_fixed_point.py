"""The fixed-point numbers of the decode kernel for one query head per KV head: 24 bits, rounded to the nearest."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import test_gpu_parity as T                                              # noqa: E402  (helpers only)

mq = T.mq


@pytest.mark.parametrize("e,G", [(0, 64), (1, 32), (2, 64)])
def test_weights_are_not_rounded_to_one_side(mq, ref, e, G):
    """Softmax weights within a factor of two of each other (the upper half of the fixed-point range) on values code * 1 + 0:
    the output is a mean of the codes, and its signed relative error, averaged over 512 rows x 128 dims, shows a one-sided
    rounding.  One unit of the fixed-point weights is 2^-24 to 2^-23 of them: half a unit too much, as odd weights would be
    with +0.5 in binary32, is 4e-8.  The binary32 sums err by some 3e-8 a row, either way: 1e-9 in the mean of 512."""
    rng = np.random.default_rng(77 + e)
    B, H, N, C = 8, 64, 64, 6
    bits = (2, 4, 8)[e]
    cfg, rcfg = T._cfgs(mq, ref, B, H, H, N, G, (2, 4, 8, 16), 0)
    K = (rng.standard_normal((B, H, C * N, 128)) * 0.05).astype(np.float16)
    V = rng.integers(192 if bits == 8 else 0, 2 ** bits, (B, H, C * N, 128)).astype(np.float16)   # 8 bits: the kernel's codes are minus 128
    V[..., ::G] = 0; V[..., 1::G] = 2 ** bits - 1                        # every group: zero 0, scale 1
    q = (rng.standard_normal((B, H, 128)) * 0.5).astype(np.float16)
    expert = np.full((B * H, C), e, np.uint8)
    (arena, used, off, status), (arena_ref, used_ref, off_ref, st_ref) = T._pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert)
    want = ref.decode_attn(rcfg, q, arena_ref, off_ref, expert, C, None, None, 0, 1 / math.sqrt(128))
    out = torch.full((B, H, 128), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(mq.decode_workspace_bytes(cfg, C), dtype=torch.uint8, device="cuda")
    mq.decode_attn(cfg, T._dev(q), arena, off, T._dev(expert), C, None, None, 0, 1 / math.sqrt(128), out, ws)
    torch.cuda.synchronize()
    rel = out.cpu().numpy().astype(np.float64)[..., 2:G] / want[..., 2:G] - 1.0
    assert abs(rel.mean()) <= 1e-8 and np.abs(rel).max() <= 1e-6, (rel.mean(), np.abs(rel).max())


@pytest.mark.parametrize("H,N,G,C,tail,mix", [
    (2, 128, 64, 300, 77, (0.6, 0.3, 0.05, 0.05)),
    (1, 256, 32, 160, 3, (0.6, 0.3, 0.05, 0.05)),
    (3, 64, 64, 500, 0, (1, 0, 0, 0)),
    (2, 128, 32, 280, 0, (0, 1, 0, 0)),
    (2, 128, 64, 260, 50, (0, 0, 1, 0)),
    (2, 32, 64, 1000, 9, (0.6, 0.3, 0.05, 0.05)),     # units of several chunks
])
def test_long_rows(mq, ref, H, N, G, C, tail, mix):
    """Rows of 32k to 41k tokens.  A score errs by 2^-25 of the largest query entry times the keys' absolute sum (some 1e-6 of a
    score's spread), a weight by 2^-25 to 2^-24, exp2 by 2^-24, the binary32 sums of 300 units by a few 2^-24, all either way:
    6e-7 to 1.3e-6 of a row's largest output.  Fixed-point numbers of 21 bits give 1.8e-6 to 6.7e-6 on these rows."""
    rng = np.random.default_rng(C)
    expert = rng.choice(4, size=(H, C), p=mix).astype(np.uint8)
    err = T._attn_case(mq, ref, 1, H, H, N, G, C, tail, (2, 4, 8, 16), N + C, expert=expert)
    assert err <= 2.5e-6, err


@pytest.mark.parametrize("H,N,G,C,tail,mix", [
    (2, 128, 32, 300, 77, (0.6, 0.3, 0.05, 0.05)),
    (2, 256, 64, 130, 3, (0.6, 0.3, 0.05, 0.05)),
    (2, 64, 32, 500, 0, (1, 0, 0, 0)),                # units that end early
    (2, 192, 64, 180, 0, (0, 1, 0, 0)),
    (2, 64, 64, 520, 50, (0, 0, 1, 0)),
    (2, 32, 32, 1000, 9, (0.6, 0.3, 0.05, 0.05)),     # units of several chunks
])
def test_long_rows_per_channel(mq, ref, H, N, G, C, tail, mix):
    """Keys quantised per channel.  q * scale of a token group is held to 2^-22 (two fp16 numbers), its products with the codes are
    summed with 24 bits: a few 1e-7 of a score's absolute sum, as binary32 multiply-adds would err; the rest as above.  One fp16
    number for q * scale, or codes in the lowest bits of their mantissas, give 5e-5 and more."""
    rng = np.random.default_rng(C + G)
    expert = rng.choice(4, size=(H, C), p=mix).astype(np.uint8)
    err = T._attn_case(mq, ref, 1, H, H, N, G, C, tail, (2, 4, 8, 16), N + C, expert=expert, kpc=1)
    assert err <= 5e-6, err
