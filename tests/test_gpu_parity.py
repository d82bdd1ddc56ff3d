"""GPU parity: the HIP library (through its C ABI) against the CPU oracle, element by element.

Routing decisions, vote counts, offsets and packed bytes must be bit-exact; attention must
stay within 2e-3 max-norm relative error per output row against the fp64 oracle.
"""
import dataclasses
import math
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ATTN_TOL = 2e-3


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu-case] {request.node.nodeid}", file=sys.stderr, flush=True)
    yield


@pytest.fixture(scope="module")
def mq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_07533_amd import binding
    binding.lib()
    return binding


def _cfgs(mq, ref, B, Hq, Hkv, N, G, bits, freeze, kpc=0):
    return (mq.Cfg(B, Hq, Hkv, 128, N, G, bits, freeze, kpc), ref.RefCfg(B, Hq, Hkv, 128, N, G, bits, freeze, kpc))


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _rand_kv(rng, B, Hkv, S, outliers=True):
    K = rng.standard_normal((B, Hkv, S, 128), dtype=np.float32)
    if outliers:
        for u in range(B * Hkv):
            K[u // Hkv, u % Hkv][:, rng.choice(128, 4, replace=False)] *= 10
    V = rng.standard_normal((B, Hkv, S, 128), dtype=np.float32)
    return K.astype(np.float16), V.astype(np.float16)


# ----------------------------------------------------------------------------------------------
# routing
# ----------------------------------------------------------------------------------------------

@pytest.mark.parametrize("B,Hkv,N,C,M,freeze,std,use_bias", [
    (1, 8, 64, 32, 4, 1, 0.02, False),      # the tiny workload's shape
    (2, 3, 32, 5, 3, 0, 0.3, True),
    (1, 2, 128, 7, 4, 2, 0.3, False),
    (1, 1, 256, 3, 8, 1, 0.2, True),
    (1, 2, 96, 4, 1, 0, 0.3, False),        # one expert; chunk not a multiple of 64
    (2, 2, 160, 3, 5, 1, 0.5, False),       # two LDS slabs with a ragged second one
    (1, 4, 128, 6, 2, 0, 1.0, True),
    (2, 2, 16, 9, 4, 1, 0.3, False),        # the small chunks of Table 3's sweep
    (1, 3, 8, 21, 4, 1, 0.3, True),
])
def test_route_bit_exact(mq, ref, B, Hkv, N, C, M, freeze, std, use_bias):
    rng = np.random.default_rng(N * 100 + M)
    bits = ([16, 2, 4, 8, 2, 4, 8, 16])[:M]
    cfg, rcfg = _cfgs(mq, ref, B, Hkv, Hkv, N, 64, bits, freeze)
    S = C * N + 11
    K, _ = _rand_kv(rng, B, Hkv, S)
    W1 = (rng.standard_normal((128, M)) * std).astype(np.float16)
    W2 = (rng.standard_normal((128, M)) * std).astype(np.float16)
    W3 = (rng.standard_normal((M, M)) * max(std, 0.2)).astype(np.float16)
    bias = (rng.standard_normal(M) * 0.05).astype(np.float32) if use_bias else None
    e_ref, v_ref = ref.route_chunks(rcfg, K, 0, C, W1, W2, W3, bias)
    expert = torch.full((B * Hkv, C), 255, dtype=torch.uint8, device="cuda")
    votes = torch.full((B * Hkv, C, M), -1, dtype=torch.int32, device="cuda")
    mq.route_chunks(cfg, _dev(K), 0, C, _dev(W1), _dev(W2), _dev(W3), None if bias is None else _dev(bias), expert, votes)
    torch.cuda.synchronize()
    assert np.array_equal(votes.cpu().numpy(), v_ref)
    assert np.array_equal(expert.cpu().numpy(), e_ref)
    # sub-range call without votes leaves the other entries alone
    if C >= 3:
        e2 = torch.full((B * Hkv, C), 255, dtype=torch.uint8, device="cuda")
        mq.route_chunks(cfg, _dev(K), C - 2, C - 1, _dev(W1), _dev(W2), _dev(W3), None if bias is None else _dev(bias), e2, None)
        e2 = e2.cpu().numpy()
        assert np.array_equal(e2[:, C - 2], e_ref[:, C - 2]) and (np.delete(e2, C - 2, 1) == 255).all()


def test_route_strided_and_ties(mq, ref):
    """Keys stored with a padded token stride; all-zero weights (every logit ties -> expert 0)."""
    rng = np.random.default_rng(5)
    B, Hkv, N, C, M = 1, 2, 64, 4, 4
    cfg, rcfg = _cfgs(mq, ref, B, Hkv, Hkv, N, 32, (2, 4, 8, 16), 0)
    big = rng.standard_normal((B, Hkv, C * N, 256), dtype=np.float32).astype(np.float16)
    Kd = _dev(big)[..., :128]                                    # token stride 256 elements
    Kh = big[..., :128]
    W = [(rng.standard_normal(s) * 0.3).astype(np.float16) for s in [(128, M), (128, M), (M, M)]]
    e_ref, v_ref = ref.route_chunks(rcfg, Kh, 0, C, *W)
    expert = torch.zeros((B * Hkv, C), dtype=torch.uint8, device="cuda")
    votes = torch.zeros((B * Hkv, C, M), dtype=torch.int32, device="cuda")
    mq.route_chunks(cfg, Kd, 0, C, *[_dev(w) for w in W], None, expert, votes)
    assert np.array_equal(votes.cpu().numpy(), v_ref) and np.array_equal(expert.cpu().numpy(), e_ref)
    Z = [np.zeros(s, np.float16) for s in [(128, M), (128, M), (M, M)]]
    mq.route_chunks(cfg, Kd, 0, C, *[_dev(w) for w in Z], None, expert, votes)
    assert (expert.cpu().numpy() == 0).all() and (votes.cpu().numpy()[..., 0] == N).all()


def _persistent_chunks(M, N, chunks):
    """More long chunks than the kernel for few of them takes (a wavefront per 64 tokens): the persistent one."""
    return N <= 64 or chunks > (4 if N <= 128 or M <= 2 else 3) * torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("M,N,C", [(2, 64, 80), (3, 32, 300), (4, 128, 70), (4, 160, 50), (4, 8, 700), (5, 64, 90), (8, 96, 66), (8, 256, 50),
                                   (4, 96, 9), (8, 256, 5)])            # the last two: few chunks
@pytest.mark.parametrize("kind", ["near", "tied", "small", "large", "zero_rows"])
def test_route_close_decisions(mq, ref, kind, M, N, C):
    """Logits that differ by a few ulps, or not at all, in some or all tokens: decisions and votes still equal the sums in order."""
    B, Hkv = 2, 8
    assert _persistent_chunks(M, N, C * B * Hkv) == (N <= 64 or C >= 50)
    rng = np.random.default_rng(M * N + len(kind))
    cfg, rcfg = _cfgs(mq, ref, B, Hkv, Hkv, N, 64, ([16, 2, 4, 8, 2, 4, 8, 16])[:M], 0)
    K, _ = _rand_kv(rng, B, Hkv, C * N)
    W1, W2 = ((rng.standard_normal((128, M)) * 0.1).astype(np.float16) for _ in range(2))
    W3 = np.repeat((rng.standard_normal((M, 1)) * 0.3).astype(np.float16), M, 1)
    bias = None
    if kind == "near":                                            # columns of W3 one ulp apart
        W3 = (W3.view(np.uint16) + rng.integers(0, 2, (M, M)).astype(np.uint16)).view(np.float16)
    elif kind == "small":                                         # subnormal weights and keys
        W1, W2, K = W1 * np.float16(1e-5), W2 * np.float16(1e-5), K * np.float16(1e-4)
        W3 = (rng.standard_normal((M, M)) * 1e-4).astype(np.float16)
        bias = (rng.standard_normal(M) * 1e-20).astype(np.float32)
    elif kind == "large":
        K = (K * np.float16(800)).clip(-65504, 65504); W1 = W1 * np.float16(100)
        W3 = (rng.standard_normal((M, M)) * 100).astype(np.float16)
    elif kind == "zero_rows":
        K[:, :, ::3] = 0; K[:, :, 5::7] *= np.float16(1e-3)
        bias = np.repeat(np.float32(0.1), M)
    e_ref, v_ref = ref.route_chunks(rcfg, K, 0, C, W1, W2, W3, bias)
    expert = torch.full((B * Hkv, C), 255, dtype=torch.uint8, device="cuda")
    votes = torch.full((B * Hkv, C, M), -1, dtype=torch.int32, device="cuda")
    mq.route_chunks(cfg, _dev(K), 0, C, _dev(W1), _dev(W2), _dev(W3), None if bias is None else _dev(bias), expert, votes)
    torch.cuda.synchronize()
    assert np.array_equal(votes.cpu().numpy(), v_ref)
    assert np.array_equal(expert.cpu().numpy(), e_ref)


@pytest.mark.parametrize("M,N,C", [(1, 64, 20), (2, 64, 160), (4, 32, 300), (4, 128, 9), (5, 64, 90), (8, 96, 66)])
@pytest.mark.parametrize("kind", ["keys", "weights", "w3", "bias"])
def test_route_infinities_and_nan(mq, ref, kind, M, N, C):
    """A NaN logit is never the larger one, on either path; infinities and NaN in keys and weights reach the logits."""
    B, Hkv = 2, 8
    rng = np.random.default_rng(M * N + len(kind))
    cfg, rcfg = _cfgs(mq, ref, B, Hkv, Hkv, N, 64, ([16, 2, 4, 8, 2, 4, 8, 16])[:M], 0)
    K, _ = _rand_kv(rng, B, Hkv, C * N)
    W = [(rng.standard_normal(s) * 0.2).astype(np.float16) for s in ((128, M), (128, M), (M, M))]
    bias = (rng.standard_normal(M) * 0.05).astype(np.float32)
    for value in (np.nan, np.inf, -np.inf):
        k, w, b = K.copy(), [x.copy() for x in W], bias.copy()
        if kind == "keys":
            k.reshape(-1)[rng.integers(0, k.size, k.size // 400)] = value
        elif kind == "weights":
            w[1][77, M - 1] = value
        elif kind == "w3":
            w[2][0, M // 2] = value
        else:
            b[M // 2] = value
        with np.errstate(all="ignore"):
            e_ref, v_ref = ref.route_chunks(rcfg, k, 0, C, *w, b)
        expert = torch.full((B * Hkv, C), 255, dtype=torch.uint8, device="cuda")
        votes = torch.full((B * Hkv, C, M), -1, dtype=torch.int32, device="cuda")
        mq.route_chunks(cfg, _dev(k), 0, C, *[_dev(x) for x in w], _dev(b), expert, votes)
        torch.cuda.synchronize()
        assert np.array_equal(votes.cpu().numpy(), v_ref) and np.array_equal(expert.cpu().numpy(), e_ref), value


def _twin_router(rng, M, share, K):
    """Experts 0 and 1 alike but for dim 127 and ahead of the others; that dim is zero in `share` of the tokens, which tie."""
    W1, W2 = ((rng.standard_normal((128, M)) * 0.1).astype(np.float16) for _ in range(2))
    W1[:127, 1] = W1[:127, 0]; W2[:127, 1] = W2[:127, 0]
    W3 = (rng.standard_normal((M, M)) * 0.02).astype(np.float16)
    W3[:, :2] = 0; W3[0, 0] = W3[1, 1] = 2
    bias = np.zeros(M, np.float32); bias[:2] = 4
    K[..., 127][rng.random(K.shape[:3]) < share] = 0
    return W1, W2, W3, bias


@pytest.mark.parametrize("M,N,C", [(2, 64, 80), (2, 64, 160), (4, 128, 70), (4, 8, 700), (5, 64, 90), (8, 32, 200), (8, 256, 64),
                                   (2, 128, 5), (3, 192, 5), (4, 96, 9), (5, 256, 3), (8, 128, 32)])    # few chunks: a wavefront per 64 tokens
@pytest.mark.parametrize("share", [0.02, 0.2, 0.6])
def test_route_some_tokens_tie(mq, ref, share, M, N, C):
    """None to most tokens of a window of 64 tie: settled four or eight at a time, in one pass or several, or a token per lane."""
    B, Hkv = 2, 8
    rng = np.random.default_rng(M * N + int(100 * share))
    cfg, rcfg = _cfgs(mq, ref, B, Hkv, Hkv, N, 64, ([16, 2, 4, 8, 2, 4, 8, 16])[:M], 0)
    K, _ = _rand_kv(rng, B, Hkv, C * N)
    W1, W2, W3, bias = _twin_router(rng, M, share, K)
    e_ref, v_ref = ref.route_chunks(rcfg, K, 0, C, W1, W2, W3, bias)
    expert = torch.full((B * Hkv, C), 255, dtype=torch.uint8, device="cuda")
    votes = torch.full((B * Hkv, C, M), -1, dtype=torch.int32, device="cuda")
    mq.route_chunks(cfg, _dev(K), 0, C, _dev(W1), _dev(W2), _dev(W3), _dev(bias), expert, votes)
    torch.cuda.synchronize()
    assert np.array_equal(votes.cpu().numpy(), v_ref) and np.array_equal(expert.cpu().numpy(), e_ref)


@pytest.mark.parametrize("N", [32, 128])
def test_route_one_expert_reads_no_keys(mq, N):
    """One expert: the decision needs no sums, so a large call takes a fraction of what one with four experts does (a tenth; half allowed)."""
    B, Hkv, C = 1, 16, 1 << 16
    C //= N
    K = torch.zeros((B, Hkv, C * N, 128), dtype=torch.float16, device="cuda")
    expert = torch.full((Hkv, C), 255, dtype=torch.uint8, device="cuda")
    us = {}
    for M in (1, 4):
        cfg = mq.Cfg(B, Hkv, Hkv, 128, N, 32, (16, 2, 4, 8)[:M], 0, 0)
        votes = torch.full((Hkv, C, M), -1, dtype=torch.int32, device="cuda")
        W = [torch.zeros(s, dtype=torch.float16, device="cuda") for s in ((128, M), (128, M), (M, M))]
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                mq.route_chunks(cfg, K, 0, C, *W, None, expert, votes)
            b.record(); torch.cuda.synchronize()
            us[M] = min(us.get(M, math.inf), a.elapsed_time(b) * 50)
        assert bool((expert == 0).all()) and bool((votes[..., 0] == N).all())
    assert us[1] < us[4] / 2, us


def _subnormal_twins(rng, kind, B, Hkv, S, M):
    """Experts 0 and 1 with the same sums from the same products in other places: the second half of a row repeats the first, and
    expert 1's weights are expert 0's with some dims d and d + 64 exchanged.  One product is far larger than its operands' subnormal
    partners in the others, so that little of those is left where a subnormal operand counts with the smallest normal exponent."""
    ints = lambda *shape: rng.integers(1, 4, shape) * rng.choice([-1.0, 1.0], shape) * 2.0 ** -24
    if kind == "keys":                                            # one weight of 8 among weights of 0.01
        x, w = ints(B, Hkv, S, 64), rng.standard_normal(128) * 0.01
        x[..., 63] = np.sign(x[..., 63]) * 2.0 ** -24; w[63] = 8
    else:                                                         # weights: one key of 8 among keys of 0.01
        x, w = rng.standard_normal((B, Hkv, S, 64)) * 0.01, ints(128)
        x[..., 63] = 8; w[63] = 2.0 ** -24; w[127] = 0
    x, w = x.astype(np.float16), w.astype(np.float16)
    W1 = np.zeros((128, M), np.float16)
    W1[:, 0] = W1[:, 1] = w
    for d in np.flatnonzero(rng.random(64) < 0.5):
        W1[[d, 64 + d], 1] = W1[[64 + d, d], 1]
    W3 = np.zeros((M, M), np.float16); W3[0, 0] = W3[1, 1] = 1
    return np.concatenate([x, x], -1), W1, W1.copy(), W3


@pytest.mark.parametrize("M,N,C", [(2, 64, 160), (4, 32, 300), (4, 128, 5), (5, 64, 90), (8, 128, 70)])
@pytest.mark.parametrize("kind", ["keys", "weights"])
def test_route_subnormal_operands(mq, ref, kind, M, N, C):
    """Sums of subnormal keys or weights, which the matrix core cuts short: two experts tie but for the order of their sums."""
    B, Hkv = 2, 8
    rng = np.random.default_rng(M * N)
    cfg, rcfg = _cfgs(mq, ref, B, Hkv, Hkv, N, 64, ([16, 2, 4, 8, 2, 4, 8, 16])[:M], 0)
    K, W1, W2, W3 = _subnormal_twins(rng, kind, B, Hkv, C * N, M)
    e_ref, v_ref = ref.route_chunks(rcfg, K, 0, C, W1, W2, W3, None)
    expert = torch.full((B * Hkv, C), 255, dtype=torch.uint8, device="cuda")
    votes = torch.full((B * Hkv, C, M), -1, dtype=torch.int32, device="cuda")
    mq.route_chunks(cfg, _dev(K), 0, C, _dev(W1), _dev(W2), _dev(W3), None, expert, votes)
    torch.cuda.synchronize()
    assert np.array_equal(votes.cpu().numpy(), v_ref) and np.array_equal(expert.cpu().numpy(), e_ref)


# ----------------------------------------------------------------------------------------------
# quantise + pack
# ----------------------------------------------------------------------------------------------

def _pack_both(mq, ref, cfg, rcfg, K, V, c0, c1, expert, start=0, slack=0):
    BH, Ccap = expert.shape
    cap = mq.arena_upper_bound(cfg, BH * (c1 - c0)) + ((start + 255) // 256) * 256 + slack
    arena_ref = np.zeros(cap, np.uint8); used_ref = np.array([start], np.uint64); off_ref = np.zeros((BH, Ccap), np.uint64)
    st_ref = ref.quantize_pack(rcfg, K, V, c0, c1, expert, arena_ref, used_ref, off_ref)
    arena = torch.zeros(cap, dtype=torch.uint8, device="cuda")
    used = torch.tensor([start], dtype=torch.int64, device="cuda")
    off = torch.zeros((BH, Ccap), dtype=torch.int64, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    mq.quantize_pack(cfg, _dev(K), _dev(V), c0, c1, _dev(expert), arena, used, off, status)
    torch.cuda.synchronize()
    return (arena, used, off, status), (arena_ref, used_ref, off_ref, st_ref)


@pytest.mark.parametrize("B,Hkv,N,G,C", [(1, 8, 64, 32, 32), (2, 2, 128, 64, 9), (1, 3, 64, 32, 6),
                                         (1, 2, 256, 64, 5), (1, 1, 192, 32, 8), (1, 2, 64, 64, 7),
                                         (2, 3, 32, 64, 21), (1, 2, 32, 32, 10),      # the paper's default chunk size
                                         (2, 2, 16, 64, 30), (1, 2, 16, 32, 13),      # one V block of 1 or 2 slices
                                         (1, 3, 8, 64, 40), (1, 2, 8, 32, 17)])       # 2 bits: half a V slice, the rest zero codes
def test_pack_bit_exact(mq, ref, B, Hkv, N, G, C):
    rng = np.random.default_rng(N + G + C)
    cfg, rcfg = _cfgs(mq, ref, B, Hkv, Hkv, N, G, (2, 4, 8, 16), 1)
    K, V = _rand_kv(rng, B, Hkv, C * N + 5)
    # adversarial groups: constants, zeros of both signs, subnormals, huge range, exact ties
    K[0, 0, 0, :64] = 3.25; K[0, 0, 1, :32] = 0.0; K[0, 0, 1, 5] = -0.0
    K[0, 0, 2, :64] = (rng.standard_normal(64) * 1e-6).astype(np.float16)
    K[0, 0, 3, 0] = 65504; K[0, 0, 3, 1] = -65504
    K[0, 0, 4, :64] = np.arange(64) * 0.5
    V[0, 0, 0] = K[0, 0, 4]; V[0, 0, 1, :32] = -7.0
    expert = rng.integers(0, 4, (B * Hkv, C)).astype(np.uint8)
    expert[:, 0] = np.arange(B * Hkv) % 4                         # every bit-width sees the adversarial rows
    (arena, used, off, status), (arena_ref, used_ref, off_ref, st_ref) = _pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert, start=300)
    assert st_ref == 0 and int(status.item()) == 0
    assert int(used.item()) == int(used_ref[0])
    assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    got = arena.cpu().numpy()
    bad = np.nonzero(got != arena_ref)[0]
    assert bad.size == 0, f"{bad.size} bytes differ, first at {bad[:5]}"


@pytest.mark.parametrize("G", [32, 64])
def test_pack_arbitrary_finite_halves(mq, ref, G):
    """Every finite fp16 bit pattern, both signs, subnormals and the largest magnitudes side by side in one group:
    ranges whose scale rounds up by a whole fp16 step, groups spanning 40 binades, near-constant groups.  The
    kernel takes no clamp and no conversion for the codes (the rounding is an addition, the words are sums of bit
    patterns), so one code outside [0, qmax] anywhere would carry into its neighbour and show up here."""
    rng = np.random.default_rng(1000 + G)
    B, Hkv, N, C = 1, 4, 64, 12
    cfg, rcfg = _cfgs(mq, ref, B, Hkv, Hkv, N, G, (2, 4, 8, 16), 0)
    S = C * N

    def halves(shape):
        bits = rng.integers(0, 1 << 16, shape, dtype=np.uint16)
        bits[(bits & 0x7C00) == 0x7C00] &= 0xBFFF                 # no Inf / NaN: clear one exponent bit
        return bits.view(np.float16)
    K, V = halves((B, Hkv, S, 128)), halves((B, Hkv, S, 128))
    # narrow groups: a few ulps around one value, so that (x - min) / scale lands on and next to .5 ties
    base = halves((B, Hkv, S // 2, 128 // G, 1)).astype(np.float32)
    step = np.abs(base) * 2.0 ** -10 + 2.0 ** -24
    K[:, :, : S // 2] = (base + step * rng.integers(0, 9, (B, Hkv, S // 2, 128 // G, G))).reshape(B, Hkv, S // 2, 128).astype(np.float16)
    K[~np.isfinite(K)] = 0
    expert = (np.arange(B * Hkv * C).reshape(B * Hkv, C) % 3).astype(np.uint8)   # 2, 4 and 8 bits
    (arena, used, off, status), (arena_ref, used_ref, off_ref, st_ref) = _pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert)
    assert st_ref == 0 and int(status.item()) == 0 and int(used.item()) == int(used_ref[0])
    bad = np.nonzero(arena.cpu().numpy() != arena_ref)[0]
    assert bad.size == 0, f"{bad.size} bytes differ, first at {bad[:5]}"


def test_pack_subrange_append_and_status(mq, ref):
    """Chunks appended by a second call land after the first; capacity and bad ids set the status word."""
    rng = np.random.default_rng(77)
    B, Hkv, N, G, C = 1, 3, 64, 64, 6
    cfg, rcfg = _cfgs(mq, ref, B, Hkv, Hkv, N, G, (2, 4, 8, 16), 1)
    K, V = _rand_kv(rng, B, Hkv, C * N)
    expert = rng.integers(0, 4, (B * Hkv, C)).astype(np.uint8)
    cap = mq.arena_upper_bound(cfg, B * Hkv * C)
    arena_ref = np.zeros(cap, np.uint8); used_ref = np.zeros(1, np.uint64); off_ref = np.zeros((B * Hkv, C), np.uint64)
    arena = torch.zeros(cap, dtype=torch.uint8, device="cuda"); used = torch.zeros(1, dtype=torch.int64, device="cuda")
    off = torch.zeros((B * Hkv, C), dtype=torch.int64, device="cuda"); status = torch.zeros(1, dtype=torch.int32, device="cuda")
    Kd, Vd, ed = _dev(K), _dev(V), _dev(expert)
    for c0, c1 in [(0, 4), (4, 5), (5, 6)]:
        assert ref.quantize_pack(rcfg, K, V, c0, c1, expert, arena_ref, used_ref, off_ref) == 0
        mq.quantize_pack(cfg, Kd, Vd, c0, c1, ed, arena, used, off, status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and int(used.item()) == int(used_ref[0])
    assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    assert np.array_equal(arena.cpu().numpy(), arena_ref)
    # capacity exceeded: status -3, nothing written
    small = torch.zeros(int(used_ref[0]) - 256, dtype=torch.uint8, device="cuda")
    used2 = torch.zeros(1, dtype=torch.int64, device="cuda"); off2 = torch.full((B * Hkv, C), 77, dtype=torch.int64, device="cuda")
    mq.quantize_pack(cfg, Kd, Vd, 0, C, ed, small, used2, off2, status)
    torch.cuda.synchronize()
    assert int(status.item()) == mq.E_ARENA and int(used2.item()) == 0
    assert (off2 == 77).all().item() and not small.any().item()
    # sticky status: the next call is a no-op
    mq.quantize_pack(cfg, Kd, Vd, 0, C, ed, arena, used2, off2, status)
    torch.cuda.synchronize()
    assert int(status.item()) == mq.E_ARENA and int(used2.item()) == 0
    # an expert index >= M
    bad = expert.copy(); bad[1, 2] = 4
    status.zero_()
    mq.quantize_pack(cfg, Kd, Vd, 0, C, _dev(bad), arena, used2, off2, status)
    torch.cuda.synchronize()
    assert int(status.item()) == mq.E_INVAL and int(used2.item()) == 0


@pytest.mark.parametrize("BH", [700, 1500])           # more rows than workgroups resident at once; above 1024: the one-workgroup plan
def test_pack_status_with_many_rows(mq, ref, BH):
    """An undersized arena with many (sequence, KV head) rows: every workgroup of the plan must reach the same
    verdict, whenever it starts: status -3, no offset, no arena byte, arena_used unchanged; then the same
    call on a large enough arena equals the oracle."""
    rng = np.random.default_rng(BH)
    N, G, C = 64, 64, 17
    cfg, rcfg = _cfgs(mq, ref, BH, 1, 1, N, G, (2, 4, 8, 16), 0)
    K = rng.standard_normal((BH, 1, C * N, 128), dtype=np.float32).astype(np.float16)
    V = rng.standard_normal((BH, 1, C * N, 128), dtype=np.float32).astype(np.float16)
    expert = rng.integers(0, 4, (BH, C)).astype(np.uint8)
    need = int(sum(ref.chunk_block_bytes(rcfg, (2, 4, 8, 16)[e]) for e in expert.ravel()))
    Kd, Vd, ed = _dev(K), _dev(V), _dev(expert)
    small = torch.zeros(need - 256, dtype=torch.uint8, device="cuda")
    used = torch.full((1,), 0, dtype=torch.int64, device="cuda"); status = torch.zeros(1, dtype=torch.int32, device="cuda")
    off = torch.full((BH, C), 77, dtype=torch.int64, device="cuda")
    for _ in range(3):                                                  # the verdict may not depend on timing
        status.zero_()
        mq.quantize_pack(cfg, Kd, Vd, 0, C, ed, small, used, off, status)
        torch.cuda.synchronize()
        assert int(status.item()) == mq.E_ARENA and int(used.item()) == 0
        assert (off == 77).all().item() and not small.any().item()
    status.zero_()
    arena = torch.zeros(need, dtype=torch.uint8, device="cuda")
    mq.quantize_pack(cfg, Kd, Vd, 0, C, ed, arena, used, off, status)
    torch.cuda.synchronize()
    arena_ref = np.zeros(need, np.uint8); used_ref = np.zeros(1, np.uint64); off_ref = np.zeros((BH, C), np.uint64)
    assert ref.quantize_pack(rcfg, K, V, 0, C, expert, arena_ref, used_ref, off_ref) == 0
    assert int(status.item()) == 0 and int(used.item()) == int(used_ref[0]) == need
    assert np.array_equal(off.cpu().numpy().astype(np.uint64), off_ref)
    assert np.array_equal(arena.cpu().numpy(), arena_ref)


# ----------------------------------------------------------------------------------------------
# decode attention
# ----------------------------------------------------------------------------------------------

def _attn_case(mq, ref, B, Hq, Hkv, N, G, C, T, bits, seed, scale=None, expert=None, freeze=1, kpc=0):
    rng = np.random.default_rng(seed)
    cfg, rcfg = _cfgs(mq, ref, B, Hq, Hkv, N, G, bits, freeze, kpc)
    S = C * N + T
    K, V = _rand_kv(rng, B, Hkv, max(S, 1))
    q = rng.standard_normal((B, Hq, 128), dtype=np.float32).astype(np.float16)
    if expert is None:
        expert = rng.integers(0, len(bits), (B * Hkv, max(C, 1))).astype(np.uint8)
    scale = 1 / math.sqrt(128) if scale is None else scale
    Kt = np.zeros((B, Hkv, N, 128), np.float16); Vt = np.zeros_like(Kt)
    Kt[:, :, :T] = K[:, :, C * N:C * N + T]; Vt[:, :, :T] = V[:, :, C * N:C * N + T]
    # rows past n_tail hold junk that must not leak into the result
    Kt[:, :, T:] = np.float16(np.nan); Vt[:, :, T:] = np.float16(np.inf)
    if C > 0:
        (arena, used, off, status), (arena_ref, used_ref, off_ref, st_ref) = _pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert)
        assert np.array_equal(arena.cpu().numpy(), arena_ref)
        ed = _dev(expert)
    else:
        arena = off = ed = None; arena_ref = off_ref = None
    o_ref = ref.decode_attn(rcfg, q, arena_ref, off_ref, expert if C else None, C, Kt, Vt, T, scale)
    out = torch.full((B, Hq, 128), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(mq.decode_workspace_bytes(cfg, C), dtype=torch.uint8, device="cuda")
    ws.fill_(0xFF)                                                # workspace contents must not matter
    mq.decode_attn(cfg, _dev(q), arena, off, ed, C, _dev(Kt) if T else None, _dev(Vt) if T else None, T, scale, out, ws)
    torch.cuda.synchronize()
    o = out.cpu().numpy().astype(np.float64)
    assert np.isfinite(o).all()
    err = np.abs(o - o_ref).max(-1) / np.abs(o_ref).max(-1)
    return err.max()


@pytest.mark.parametrize("B,Hq,Hkv,N,G,C,T", [
    (1, 8, 8, 64, 32, 32, 0),        # tiny workload shape
    (1, 8, 8, 64, 32, 9, 13),
    (2, 4, 4, 128, 64, 20, 1),
    (1, 8, 2, 128, 64, 33, 127),     # GQA x4, long tail
    (1, 4, 2, 256, 64, 7, 200),      # GQA x2
    (1, 8, 1, 64, 64, 40, 31),       # GQA x8, smallest chunk
    (1, 2, 2, 192, 32, 5, 100),      # three 64-token blocks per chunk
    (2, 2, 2, 64, 64, 3, 0),
    (1, 2, 2, 192, 64, 11, 50),
    (1, 1, 1, 128, 64, 600, 5),      # more chunks than splits*64: several descriptor batches
    (1, 4, 4, 32, 64, 70, 19),       # chunks of 32 tokens (the paper's default): half tiles at 2 bits, short units at 4 bits
    (2, 2, 2, 32, 32, 33, 0),
    (1, 8, 2, 32, 64, 50, 31),       # ... with grouped queries x4
    (1, 4, 2, 32, 32, 9, 5),
    (1, 2, 2, 32, 64, 2500, 3),      # ... and several row segments (more than 1024 chunks per row)
    (1, 4, 4, 16, 64, 90, 11),       # chunks of 16 tokens: units shorter than a KiB of codes at 2 bits
    (2, 2, 2, 16, 32, 41, 0),
    (1, 8, 2, 16, 64, 70, 15),       # ... with grouped queries x4
    (1, 4, 4, 8, 64, 150, 5),        # chunks of 8 tokens: short units at 2 and 4 bits, padded V slice at 2 bits, 8-row FP16 units
    (2, 2, 2, 8, 32, 77, 7),
    (1, 8, 2, 8, 64, 120, 3),        # ... with grouped queries x4
    (1, 4, 2, 8, 32, 60, 0),
    (1, 1, 1, 8, 64, 2100, 1),       # ... and several row segments
])
def test_attention_mixed_bits(mq, ref, B, Hq, Hkv, N, G, C, T):
    err = _attn_case(mq, ref, B, Hq, Hkv, N, G, C, T, (2, 4, 8, 16), seed=C * 7 + T)
    assert err <= ATTN_TOL, err


@pytest.mark.parametrize("bits", [(2,), (4,), (8,), (16,)])
@pytest.mark.parametrize("N,G,rep", [(128, 64, 1), (64, 32, 4), (192, 32, 1), (256, 64, 2), (32, 64, 1), (32, 64, 8), (32, 32, 2),
                                     (16, 64, 1), (16, 32, 2), (16, 64, 8), (8, 64, 1), (8, 32, 1), (8, 64, 4), (8, 32, 4)])
def test_attention_single_bit_width(mq, ref, bits, N, G, rep):
    err = _attn_case(mq, ref, 1, 2 * rep, 2, N, G, 12, min(17, N - 1), bits, seed=bits[0] + N, freeze=0)
    assert err <= ATTN_TOL, err


@pytest.mark.parametrize("heavy,B,Hkv,rep,N,C,T", [
    (3, 1, 8, 1, 128, 160, 40),      # one row of 16-bit chunks among 2-bit rows: the rows have the same number of workgroups all the same
    (0, 2, 4, 1, 64, 300, 0),
    (-1, 1, 8, 1, 128, 160, 0),      # the reverse: one 2-bit row among 16-bit rows
    (5, 1, 8, 4, 256, 60, 100),      # grouped queries
    (2, 1, 40, 1, 128, 48, 7),       # the workgroups add up the rows' costs and find them too uneven: intervals
    (3, 75, 4, 1, 128, 8, 7),        # more rows than compute units, on intervals: the heavy row takes most workgroups
    (-1, 75, 4, 2, 128, 8, 0),
    (5, 1, 40, 1, 16, 410, 3),       # intervals, short chunks: 240 workgroups would leave compute units idle
])
def test_attention_rows_of_unequal_cost(mq, ref, heavy, B, Hkv, rep, N, C, T):
    """Rows whose mixes of bit-widths differ as much as they can, on even shares and on intervals of equal cost."""
    bits = (2, 4, 8, 16)
    BH = B * Hkv
    expert = np.zeros((BH, C), np.uint8)                          # 2 bits everywhere ...
    if heavy >= 0:
        expert[heavy % BH] = 3                                    # ... but one row of 16-bit chunks
    else:
        expert[:] = 3; expert[BH // 2] = 0
    expert[:, 1::7] = 1                                           # and a few 4-bit chunks in every row
    err = _attn_case(mq, ref, B, Hkv * rep, Hkv, N, 64, C, T, bits, seed=BH + C, expert=expert, freeze=0)
    assert err <= ATTN_TOL, err


@pytest.mark.parametrize("B,H,N,G,C,T,bits", [
    (1, 4, 128, 64, 21, 17, (2, 4, 8, 16)),
    (2, 2, 64, 64, 30, 0, (2, 4, 8, 16)),          # short 2-bit units
    (1, 2, 64, 32, 17, 5, (2, 4, 8, 16)),          # four token groups per 2-bit unit ... two per chunk
    (1, 2, 256, 64, 6, 200, (2, 4, 8, 16)),
    (1, 2, 32, 32, 40, 9, (2, 4, 8, 16)),          # chunks of 32 tokens
    (1, 1, 128, 32, 5, 0, (2,)), (1, 1, 128, 64, 5, 0, (4,)), (1, 1, 192, 64, 5, 3, (8,)),
])
def test_per_channel_keys(mq, ref, B, H, N, G, C, T, bits):
    """Keys quantised per channel (groups of G tokens of one dim): packed bytes bit-exact (checked inside _attn_case),
    attention within the tolerance, one query head per KV head."""
    err = _attn_case(mq, ref, B, H, H, N, G, C, T, bits, seed=N + C, freeze=0, kpc=1)
    assert err <= ATTN_TOL, err


def test_per_channel_keys_limits(mq):
    cfg = mq.Cfg(1, 8, 2, 128, 128, 64, (2, 4, 8, 16), 1, 1)             # grouped queries: pack yes, decode no
    assert mq.chunk_block_bytes(cfg, 2) == 10240 and mq.decode_workspace_bytes(mq.Cfg(1, 2, 2, 128, 128, 64, (2, 16), 1, 1), 4) > 0
    q = torch.zeros((1, 8, 128), dtype=torch.float16, device="cuda"); out = torch.zeros((1, 8, 128), dtype=torch.float32, device="cuda")
    ws = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
    Kt = torch.zeros((1, 2, 128, 128), dtype=torch.float16, device="cuda")
    with pytest.raises(mq.MoqaeError) as e:
        mq.decode_attn(cfg, q, None, None, None, 0, Kt, Kt, 5, 0.1, out, ws)
    assert e.value.code == mq.E_INVAL
    assert mq.chunk_block_bytes(mq.Cfg(1, 2, 2, 128, 32, 64, (2, 16), 1, 1), 2) == 0     # token groups must tile the chunk


@pytest.mark.parametrize("B,Hq,Hkv,Q,N,G,C,T", [
    (1, 2, 2, 4, 128, 64, 23, 50),       # four new tokens, one query head per KV head
    (2, 4, 2, 2, 64, 64, 17, 2),         # grouped queries x2, two new tokens, nothing else in the residual
    (1, 4, 1, 2, 64, 64, 9, 33),         # x4 heads x 2 tokens: eight rows per KV head; the new tokens straddle two 16-row units
    (1, 1, 1, 8, 256, 64, 5, 8),         # eight new tokens
    (1, 2, 2, 4, 32, 64, 41, 4),         # chunks of 32 tokens
    (1, 2, 2, 4, 8, 64, 37, 6),          # chunks of 8 tokens: the residual buffers hold 8 rows
    (1, 4, 2, 2, 16, 64, 29, 3),
    (1, 3, 3, 1, 128, 64, 6, 7),         # one query: the plain decode call
    (1, 2, 2, 4, 64, 64, 0, 20),         # no packed chunk yet
])
def test_attention_several_queries(mq, ref, B, Hq, Hkv, Q, N, G, C, T):
    """moqae_decode_attn_multi: Q new tokens per sequence, causal among themselves, against the oracle."""
    rng = np.random.default_rng(Q * 100 + C)
    bits = (2, 4, 8, 16)
    cfg, rcfg = _cfgs(mq, ref, B, Hq, Hkv, N, G, bits, 1)
    S = C * N + T
    K, V = _rand_kv(rng, B, Hkv, S)
    q = rng.standard_normal((B, Q, Hq, 128), dtype=np.float32).astype(np.float16)
    Kt = np.zeros((B, Hkv, N, 128), np.float16); Vt = np.zeros_like(Kt)
    Kt[:, :, :T] = K[:, :, C * N:]; Vt[:, :, :T] = V[:, :, C * N:]
    Kt[:, :, T:] = np.float16(np.nan); Vt[:, :, T:] = np.float16(np.inf)
    if C > 0:
        expert = rng.integers(0, 4, (B * Hkv, C)).astype(np.uint8)
        (arena, used, off, status), (arena_ref, used_ref, off_ref, st_ref) = _pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert)
        ed = _dev(expert)
    else:
        expert = arena = off = ed = arena_ref = off_ref = None
    scale = 1 / math.sqrt(128)
    o_ref = ref.decode_attn_multi(rcfg, q, arena_ref, off_ref, expert, C, Kt, Vt, T, scale)
    out = torch.full((B, Q, Hq, 128), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(mq.decode_workspace_bytes_multi(cfg, C, Q), dtype=torch.uint8, device="cuda"); ws.fill_(0xFF)
    mq.decode_attn_multi(cfg, _dev(q), arena, off, ed, C, _dev(Kt), _dev(Vt), T, scale, out, ws)
    torch.cuda.synchronize()
    o = out.cpu().numpy().astype(np.float64)
    assert np.isfinite(o).all()
    err = np.abs(o - o_ref).max(-1) / np.abs(o_ref).max(-1)
    assert err.max() <= ATTN_TOL, err.max()


def test_attention_degenerate_cases(mq, ref):
    # residual rows only (no packed chunk), down to a single cached token
    assert _attn_case(mq, ref, 1, 4, 2, 64, 32, 0, 1, (2, 16), seed=1) <= ATTN_TOL
    assert _attn_case(mq, ref, 2, 2, 2, 128, 64, 0, 97, (2, 16), seed=2) <= ATTN_TOL
    # one chunk, no residual
    assert _attn_case(mq, ref, 1, 2, 2, 64, 32, 1, 0, (4, 16), seed=3) <= ATTN_TOL
    # a sharp softmax (one key dominates) and a flat one
    assert _attn_case(mq, ref, 1, 2, 2, 64, 64, 8, 3, (2, 4, 8, 16), seed=4, scale=3.0) <= ATTN_TOL
    assert _attn_case(mq, ref, 1, 2, 2, 64, 64, 8, 3, (2, 4, 8, 16), seed=5, scale=0.0) <= ATTN_TOL


def test_argument_errors(mq):
    cfg = mq.Cfg(1, 2, 2, 128, 64, 32, (2, 4, 8, 16), 1)
    q = torch.zeros((1, 2, 128), dtype=torch.float16, device="cuda")
    out = torch.zeros((1, 2, 128), dtype=torch.float32, device="cuda")
    ws = torch.zeros(16, dtype=torch.uint8, device="cuda")
    Kt = torch.zeros((1, 2, 64, 128), dtype=torch.float16, device="cuda")
    with pytest.raises(mq.MoqaeError) as e:
        mq.decode_attn(cfg, q, None, None, None, 0, Kt, Kt, 5, 0.1, out, ws)
    assert e.value.code == mq.E_WORKSPACE
    # the packed layout tiles 64 tokens at a time: routing accepts a 32- or 96-token chunk, pack and decode do not
    c96 = mq.Cfg(1, 2, 2, 128, 96, 32, (2, 4, 8, 16), 1)
    assert mq.decode_workspace_bytes(c96, 4) == 0
    with pytest.raises(mq.MoqaeError) as e:
        Kt96 = torch.zeros((1, 2, 96, 128), dtype=torch.float16, device="cuda")
        mq.decode_attn(c96, q, None, None, None, 0, Kt96, Kt96, 5, 0.1, out, torch.zeros(1 << 20, dtype=torch.uint8, device="cuda"))
    assert e.value.code == mq.E_INVAL
    # grouped queries: (query heads per KV head) x (groups per row) must fit the 16 rows of a matrix-core tile
    g8 = mq.Cfg(1, 8, 1, 128, 64, 32, (2, 4, 8, 16), 1)
    assert mq.decode_workspace_bytes(g8, 4) == 0
    bad = mq.Cfg(1, 3, 2, 128, 64, 32, (2, 4, 8, 16), 1)                 # Hq not a multiple of Hkv
    assert mq.decode_workspace_bytes(bad, 4) == 0 and mq.chunk_block_bytes(bad, 2) == 0
    nofp16 = mq.Cfg(1, 2, 2, 128, 64, 32, (2, 4, 8), 1)                  # freezing needs a 16-bit expert
    W = torch.zeros((128, 3), dtype=torch.float16, device="cuda")
    with pytest.raises(mq.MoqaeError) as e:
        mq.route_chunks(nofp16, Kt, 0, 1, W, W, torch.zeros((3, 3), dtype=torch.float16, device="cuda"), None,
                        torch.zeros((2, 1), dtype=torch.uint8, device="cuda"))
    assert e.value.code == mq.E_INVAL


# ----------------------------------------------------------------------------------------------
# decode attention over a batch of sequences of different lengths
# ----------------------------------------------------------------------------------------------

def _ragged_case(mq, ref, Hq, Hkv, N, G, lens, bits=(2, 4, 8, 16), seed=0, kpc=0):
    """lens: tokens per sequence.  Every sequence's cache is packed up to its own last full chunk; the oracle is
    called per sequence (batch 1) on that sequence's slice of the tables."""
    rng = np.random.default_rng(seed)
    B = len(lens)
    Cs = [L // N for L in lens]; Ts = [L % N for L in lens]
    Cmax = max(max(Cs), 1)
    cfg, rcfg = _cfgs(mq, ref, B, Hq, Hkv, N, G, bits, 1, kpc)
    _, rcfg1 = _cfgs(mq, ref, 1, Hq, Hkv, N, G, bits, 1, kpc)
    K, V = _rand_kv(rng, B, Hkv, Cmax * N + N)
    q = rng.standard_normal((B, Hq, 128), dtype=np.float32).astype(np.float16)
    expert = rng.integers(0, len(bits), (B * Hkv, Cmax)).astype(np.uint8)
    scale = 1 / math.sqrt(128)
    Kt = np.full((B, Hkv, N, 128), np.nan, np.float16); Vt = np.full((B, Hkv, N, 128), np.inf, np.float16)
    for b in range(B):
        Kt[b, :, :Ts[b]] = K[b, :, Cs[b] * N:Cs[b] * N + Ts[b]]; Vt[b, :, :Ts[b]] = V[b, :, Cs[b] * N:Cs[b] * N + Ts[b]]
    # all Cmax chunks of every sequence are packed; a sequence only attends to its first Cs[b]
    (arena, used, off, status), (arena_ref, used_ref, off_ref, st_ref) = _pack_both(mq, ref, cfg, rcfg, K, V, 0, Cmax, expert)
    assert np.array_equal(arena.cpu().numpy(), arena_ref)
    out = torch.full((B, Hq, 128), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(mq.decode_workspace_bytes_ragged(cfg, Cmax), dtype=torch.uint8, device="cuda")
    ws.fill_(0xFF)
    nc = torch.tensor(Cs, dtype=torch.int32, device="cuda"); nt = torch.tensor(Ts, dtype=torch.int32, device="cuda")
    mq.decode_attn_ragged(cfg, _dev(q), arena, off, _dev(expert), nc, Cmax, _dev(Kt), _dev(Vt), nt, scale, out, ws)
    torch.cuda.synchronize()
    o = out.cpu().numpy().astype(np.float64)
    worst = 0.0
    for b in range(B):
        if lens[b] == 0:
            assert (o[b] == 0).all()                              # a sequence without tokens: zeros
            continue
        rows = slice(b * Hkv, (b + 1) * Hkv)
        o_ref = ref.decode_attn(rcfg1, q[b:b + 1], arena_ref, off_ref[rows], expert[rows], Cs[b],
                                np.nan_to_num(Kt[b:b + 1], nan=0.0, posinf=0.0), np.nan_to_num(Vt[b:b + 1], nan=0.0, posinf=0.0),
                                Ts[b], scale)
        assert np.isfinite(o[b]).all()
        worst = max(worst, (np.abs(o[b] - o_ref[0]).max(-1) / np.abs(o_ref[0]).max(-1)).max())
    return worst


@pytest.mark.parametrize("Hq,Hkv,N,G,lens", [
    (4, 4, 64, 32, [64 * 30 + 5, 17, 64 * 7, 0, 64 * 12 + 63, 1]),          # long, residual only, whole chunks, empty, one token
    (8, 2, 128, 64, [128 * 40 + 100, 128 * 3, 90, 128 * 17 + 1]),           # grouped queries x4
    (2, 2, 256, 64, [256 * 9 + 255, 256, 255, 256 * 4]),
    (2, 1, 64, 64, [64 * 300, 64 * 2 + 1, 5]),                              # grouped queries x2, one row much longer than the rest
    (3, 3, 128, 64, [0, 0, 77]),                                            # almost everything empty
    (4, 2, 32, 64, [32 * 50 + 7, 31, 32 * 3, 0]),                           # chunks of 32 tokens, grouped queries x2
    (2, 2, 8, 64, [8 * 200 + 7, 5, 8 * 3, 0]),                              # chunks of 8 tokens
    (4, 1, 16, 32, [16 * 90 + 15, 16, 1]),
])
def test_attention_ragged_batch(mq, ref, Hq, Hkv, N, G, lens):
    err = _ragged_case(mq, ref, Hq, Hkv, N, G, lens, seed=len(lens) * 31 + N)
    assert err <= ATTN_TOL, err


@pytest.mark.parametrize("H,N,G,lens", [
    (2, 128, 64, [128 * 33 + 100, 128 * 3, 90, 0, 128 * 17 + 1]),
    (3, 64, 32, [64 * 70 + 5, 17, 64 * 7, 64 * 12 + 63]),
    (2, 32, 32, [32 * 50 + 7, 31, 32 * 3, 0]),                              # chunks of 32 tokens
    (1, 256, 64, [256 * 9 + 255, 256, 255]),
])
def test_per_channel_keys_ragged_batch(mq, ref, H, N, G, lens):
    """Keys quantised per channel in a batch of sequences of different lengths."""
    err = _ragged_case(mq, ref, H, H, N, G, lens, seed=len(lens) * 17 + N, kpc=1)
    assert err <= ATTN_TOL, err


def test_attention_ragged_equals_uniform(mq, ref):
    """With equal lengths the ragged call reproduces the uniform call (same kernels, same tickets) to rounding."""
    rng = np.random.default_rng(5)
    B, Hq, Hkv, N, G, C, T = 3, 4, 4, 128, 64, 21, 40
    cfg, rcfg = _cfgs(mq, ref, B, Hq, Hkv, N, G, (2, 4, 8, 16), 1)
    K, V = _rand_kv(rng, B, Hkv, C * N + T)
    q = _dev(rng.standard_normal((B, Hq, 128), dtype=np.float32).astype(np.float16))
    expert = rng.integers(0, 4, (B * Hkv, C)).astype(np.uint8)
    (arena, used, off, status), _ = _pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert)
    Kt = np.zeros((B, Hkv, N, 128), np.float16); Vt = np.zeros_like(Kt)
    Kt[:, :, :T] = K[:, :, C * N:]; Vt[:, :, :T] = V[:, :, C * N:]
    Ktd, Vtd, ed = _dev(Kt), _dev(Vt), _dev(expert)
    out_u = torch.zeros((B, Hq, 128), dtype=torch.float32, device="cuda"); out_r = torch.zeros_like(out_u)
    ws = torch.zeros(mq.decode_workspace_bytes_ragged(cfg, C), dtype=torch.uint8, device="cuda")
    scale = 1 / math.sqrt(128)
    mq.decode_attn(cfg, q, arena, off, ed, C, Ktd, Vtd, T, scale, out_u, ws)
    nc = torch.full((B,), C, dtype=torch.int32, device="cuda"); nt = torch.full((B,), T, dtype=torch.int32, device="cuda")
    mq.decode_attn_ragged(cfg, q, arena, off, ed, nc, C, Ktd, Vtd, nt, scale, out_r, ws)
    torch.cuda.synchronize()
    a, b = out_u.cpu().numpy(), out_r.cpu().numpy()
    assert np.abs(a - b).max() <= 1e-5 * np.abs(a).max()


# ----------------------------------------------------------------------------------------------
# the calls under HIP graph capture
# ----------------------------------------------------------------------------------------------

def test_hot_path_replays_from_a_hip_graph(mq, ref):
    """Route + pack + decode captured once into a HIP graph and replayed with new inputs in the same buffers: every
    replay must equal the eager calls on those inputs (the library clears its counters with kernels, not with
    memset nodes, and allocates nothing)."""
    rng = np.random.default_rng(11)
    B, Hq, Hkv, N, G, C, T = 2, 8, 4, 128, 64, 12, 30
    cfg, _ = _cfgs(mq, ref, B, Hq, Hkv, N, G, (2, 4, 8, 16), 1)
    M = 4
    W = [_dev((rng.standard_normal(s) * 0.3).astype(np.float16)) for s in [(128, M), (128, M), (M, M)]]
    Kd = torch.zeros((B, Hkv, C * N, 128), dtype=torch.float16, device="cuda"); Vd = torch.zeros_like(Kd)
    q = torch.zeros((B, Hq, 128), dtype=torch.float16, device="cuda")
    Kt = torch.zeros((B, Hkv, N, 128), dtype=torch.float16, device="cuda"); Vt = torch.zeros_like(Kt)
    cap = mq.arena_upper_bound(cfg, B * Hkv * C)

    def buffers():
        return dict(expert=torch.zeros((B * Hkv, C), dtype=torch.uint8, device="cuda"),
                    arena=torch.zeros(cap, dtype=torch.uint8, device="cuda"),
                    used=torch.zeros(1, dtype=torch.int64, device="cuda"),
                    off=torch.zeros((B * Hkv, C), dtype=torch.int64, device="cuda"),
                    status=torch.zeros(1, dtype=torch.int32, device="cuda"),
                    out=torch.zeros((B, Hq, 128), dtype=torch.float32, device="cuda"),
                    ws=torch.zeros(mq.decode_workspace_bytes(cfg, C), dtype=torch.uint8, device="cuda"))

    def path(b):
        b["used"].zero_()
        mq.route_chunks(cfg, Kd, 0, C, *W, None, b["expert"], None)
        mq.quantize_pack(cfg, Kd, Vd, 0, C, b["expert"], b["arena"], b["used"], b["off"], b["status"])
        mq.decode_attn(cfg, q, b["arena"], b["off"], b["expert"], C, Kt, Vt, T, 1 / math.sqrt(128), b["out"], b["ws"])

    def new_inputs(seed):
        r = np.random.default_rng(seed)
        K, V = _rand_kv(r, B, Hkv, C * N + T)
        Kd.copy_(_dev(K[:, :, :C * N])); Vd.copy_(_dev(V[:, :, :C * N]))
        Kt[:, :, :T].copy_(_dev(K[:, :, C * N:])); Vt[:, :, :T].copy_(_dev(V[:, :, C * N:]))
        q.copy_(_dev(r.standard_normal((B, Hq, 128), dtype=np.float32).astype(np.float16)))

    bg, be = buffers(), buffers()
    new_inputs(100)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        path(bg)                                                  # warm-up outside the capture (occupancy query, module load)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        path(bg)
    for rep in range(3):
        new_inputs(200 + rep)
        graph.replay()
        torch.cuda.synchronize()
        path(be)                                                  # the program's own eager work between the replays
        torch.cuda.synchronize()
        assert int(bg["status"].item()) == 0 and int(be["status"].item()) == 0
        assert torch.equal(bg["expert"], be["expert"]) and torch.equal(bg["off"], be["off"])
        n_used = int(be["used"].item())                          # beyond it the arenas hold what earlier inputs left
        assert int(bg["used"].item()) == n_used and torch.equal(bg["arena"][:n_used], be["arena"][:n_used])
        a, b = bg["out"].cpu().numpy(), be["out"].cpu().numpy()
        # attention: equal up to the order in which the wavefronts drew their units (grouped queries round their
        # weights to fp16 relative to the running maximum of the moment), far inside the 2e-3 bar
        assert np.isfinite(a).all() and np.abs(a - b).max() <= 2e-4 * np.abs(b).max()


# ----------------------------------------------------------------------------------------------
# decode steps on a plan
# ----------------------------------------------------------------------------------------------

@pytest.mark.parametrize("B,Hq,Hkv,N,G,C", [(2, 4, 4, 128, 64, 23), (1, 8, 2, 64, 32, 40), (1, 2, 2, 256, 64, 0)])
def test_attention_on_a_plan(mq, ref, B, Hq, Hkv, N, G, C):
    """moqae_decode_plan once, then several moqae_decode_attn_planned calls with a growing residual and new queries:
    each equals the oracle, and an unplanned call in between (which overwrites the plan) needs a new plan."""
    rng = np.random.default_rng(C + N)
    cfg, rcfg = _cfgs(mq, ref, B, Hq, Hkv, N, G, (2, 4, 8, 16), 1)
    K, V = _rand_kv(rng, B, Hkv, C * N + N)
    expert = rng.integers(0, 4, (B * Hkv, max(C, 1))).astype(np.uint8)
    scale = 1 / math.sqrt(128)
    if C > 0:
        (arena, used, off, status), (arena_ref, used_ref, off_ref, st_ref) = _pack_both(mq, ref, cfg, rcfg, K, V, 0, C, expert)
        ed = _dev(expert)
    else:
        arena = off = ed = None; arena_ref = off_ref = None
    ws = torch.empty(mq.decode_workspace_bytes(cfg, C), dtype=torch.uint8, device="cuda")
    ws.fill_(0xFF)
    out = torch.zeros((B, Hq, 128), dtype=torch.float32, device="cuda")
    mq.decode_plan(cfg, ed, C, ws)
    for step, T in enumerate([1, 2, 17, N // 2, N - 1]):
        q = rng.standard_normal((B, Hq, 128), dtype=np.float32).astype(np.float16)
        Kt = np.zeros((B, Hkv, N, 128), np.float16); Vt = np.zeros_like(Kt)
        Kt[:, :, :T] = K[:, :, C * N:C * N + T]; Vt[:, :, :T] = V[:, :, C * N:C * N + T]
        o_ref = ref.decode_attn(rcfg, q, arena_ref, off_ref, expert if C else None, C, Kt, Vt, T, scale)
        if step == 3:                                             # an ordinary call uses the workspace its own way
            mq.decode_attn(cfg, _dev(q), arena, off, ed, C, _dev(Kt), _dev(Vt), T, scale, out, ws)
            mq.decode_plan(cfg, ed, C, ws)
        out.fill_(float("nan"))
        mq.decode_attn(cfg, _dev(q), arena, off, ed, C, _dev(Kt), _dev(Vt), T, scale, out, ws, planned=True)
        torch.cuda.synchronize()
        o = out.cpu().numpy().astype(np.float64)
        assert np.isfinite(o).all()
        err = (np.abs(o - o_ref).max(-1) / np.abs(o_ref).max(-1)).max()
        assert err <= ATTN_TOL, (step, err)


def test_append_tail(mq, ref):
    """The new token's rows land in row n_tail of both residual buffers and nowhere else."""
    cfg, _ = _cfgs(mq, ref, 3, 8, 4, 128, 64, (2, 4, 8, 16), 1)
    g = torch.Generator(device="cuda"); g.manual_seed(3)
    Kt = torch.randn((3, 4, 128, 128), generator=g, device="cuda").half(); Vt = torch.randn((3, 4, 128, 128), generator=g, device="cuda").half()
    for n_tail in (0, 77, 127):
        kn = torch.randn((3, 4, 128), generator=g, device="cuda").half(); vn = torch.randn((3, 4, 128), generator=g, device="cuda").half()
        Kr, Vr = Kt.clone(), Vt.clone()
        Kr[:, :, n_tail] = kn; Vr[:, :, n_tail] = vn
        mq.append_tail(cfg, kn, vn, Kt, Vt, n_tail)
        torch.cuda.synchronize()
        assert torch.equal(Kt, Kr) and torch.equal(Vt, Vr)
    with pytest.raises(mq.MoqaeError):
        mq.append_tail(cfg, kn, vn, Kt, Vt, 128)
