"""GPU parity of moqae_router_loss_grad (the router fine-tuning loss of Sec. 3.3, Eq. (3)-(5), and its gradient)
against the CPU oracle (binary64 given the binary32 top-1 decision)."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import test_gpu_parity as T                                              # noqa: E402  (helpers only)

mq = T.mq
BITS = (2, 4, 8, 16)
# binary32 forward / backward per row and sums over up to ~1e5 rows added in no fixed order, against binary64:
# relative to the largest entry of each gradient array
GRAD_TOL, LOSS_TOL = 2e-4, 2e-5


@pytest.mark.parametrize("B,Hkv,S,t0,t1,M,std,use_bias,defaults", [
    (1, 8, 2048, 0, 2048, 4, 0.02, False, True),      # the tiny workload's shape, router at its initial scale
    (2, 3, 700, 13, 650, 4, 0.3, True, False),        # ragged token range, partial last tile
    (1, 2, 200, 0, 200, 3, 0.3, True, False),
    (3, 1, 130, 64, 130, 8, 0.2, False, False),
    (1, 1, 64, 0, 1, 1, 0.3, False, True),            # one row, one expert
])
def test_router_loss_grad(mq, ref, B, Hkv, S, t0, t1, M, std, use_bias, defaults):
    print(f"\n[gpu-case] train B={B} Hkv={Hkv} S={S} [{t0},{t1}) M={M}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(S + M)
    bits = BITS[:M] if M <= 4 else (2, 2, 4, 4, 8, 8, 16, 16)
    cfg, rcfg = T._cfgs(mq, ref, B, Hkv, Hkv, 64, 64, bits, 0)
    K, _ = T._rand_kv(rng, B, Hkv, S)
    W1 = (rng.standard_normal((128, M)) * std).astype(np.float16)
    W2 = (rng.standard_normal((128, M)) * std).astype(np.float16)
    W3 = (rng.standard_normal((M, M)) * (0.5 if std > 0.1 else 0.02) + (np.eye(M) if std > 0.1 else 0)).astype(np.float16)
    bias = (rng.standard_normal(M) * 0.1).astype(np.float32) if use_bias else None
    nll = rng.uniform(1.5, 3.0, B).astype(np.float32)
    pm = np.array([1.0 / b for b in bits], np.float32)
    pe = np.array([16.0 / b for b in bits], np.float32) if defaults else np.array([b / 16.0 for b in bits], np.float32)
    lam = 0.5
    l_ref, g1, g2, g3, gb = ref.router_loss_grad(rcfg, K, t0, t1, W1, W2, W3, bias, nll, pm, pe, lam)
    dev = "cuda"
    loss = torch.full((3,), 7.0, dtype=torch.float32, device=dev)              # outputs are overwritten
    dW1 = torch.full((128, M), 7.0, dtype=torch.float32, device=dev); dW2 = torch.full_like(dW1, 7.0)
    dW3 = torch.full((M, M), 7.0, dtype=torch.float32, device=dev); db = torch.full((M,), 7.0, dtype=torch.float32, device=dev)
    mq.router_loss_grad(cfg, T._dev(K), t0, t1, T._dev(W1), T._dev(W2), T._dev(W3), None if bias is None else T._dev(bias),
                        T._dev(nll), None if defaults else pm, None if defaults else pe, lam, loss, dW1, dW2, dW3, db)
    torch.cuda.synchronize()
    l = loss.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(l - l_ref) <= LOSS_TOL * np.abs(l_ref).max()), (l, l_ref)
    for name, g, r in (("dW1", dW1, g1), ("dW2", dW2, g2), ("dW3", dW3, g3), ("dbias", db, gb)):
        got = g.cpu().numpy().astype(np.float64)
        scale = max(np.abs(r).max(), 1e-30)
        assert np.abs(got - r).max() <= GRAD_TOL * scale, (name, np.abs(got - r).max() / scale)


@pytest.mark.parametrize("Hkv,S,t0,M,pad", [
    (70, 2000, 0, 4, 0),            # more tiles than wavefronts: several tiles each, the last of a row partly empty
    (3, 65, 0, 5, 0),               # a tile of one row; two operand sets (more than four experts)
    (5, 191, 1, 2, 8),              # rows 136 elements apart
    (1, 63, 0, 7, 0),
])
def test_router_loss_grad_tiles(mq, ref, Hkv, S, t0, M, pad):
    """Edges of the 64-row tiles, strided rows, one and two operand sets of the weight gradient's matrix products."""
    rng = np.random.default_rng(S * 10 + M)
    bits = (2, 4, 8, 16, 2, 4, 8, 16)[:M]
    cfg, rcfg = T._cfgs(mq, ref, 1, Hkv, Hkv, 64, 64, bits, 0)
    K, _ = T._rand_kv(rng, 1, Hkv, S)
    W1, W2 = ((rng.standard_normal((128, M)) * 0.1).astype(np.float16) for _ in range(2))
    W3 = (rng.standard_normal((M, M)) * 0.5).astype(np.float16)
    nll = np.array([2.0], np.float32)
    pm, pe = np.array([1.0 / b for b in bits], np.float32), np.array([16.0 / b for b in bits], np.float32)
    want = ref.router_loss_grad(rcfg, K, t0, S, W1, W2, W3, None, nll, pm, pe, 0.3)
    Kd = torch.full((1, Hkv, S, 128 + pad), float("nan"), dtype=torch.float16, device="cuda")   # what lies between the rows is not read
    Kd[..., :128] = T._dev(K)
    got = [torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in ((3,), (128, M), (128, M), (M, M), (M,))]
    mq.router_loss_grad(cfg, Kd[..., :128], t0, S, T._dev(W1), T._dev(W2), T._dev(W3), None, T._dev(nll), None, None, 0.3, *got)
    torch.cuda.synchronize()
    l = got[0].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(l - want[0]) <= LOSS_TOL * np.abs(want[0]).max()), (l, want[0])
    _check_columns(("dW1", "dW2", "dW3", "dbias"), got[1:], want[1:])


# Every column (expert) by itself, 2-norm.  The binary32 sums of 128 products that a value is made of err by about
# sqrt(128) * 2^-24 = 7e-7 of their terms' norm (127 * 2^-24 = 7.6e-6 of their absolute sum at the worst), and a few such sums
# are multiplied with each other; the split of a value into two fp16 numbers adds 2^-22 = 2.4e-7.  A value cut to its first
# fp16 number errs by 1.4e-4, a column lost to another's scale by all of it.
COLUMN_TOL = 1e-5


def _check_columns(names, got, want):
    for name, g, r in zip(names, got, want):
        err = np.linalg.norm(g.cpu().numpy().astype(np.float64) - r, axis=0) / np.maximum(np.linalg.norm(r, axis=0), 1e-300)
        assert np.max(err) <= COLUMN_TOL, (name, err)


@pytest.mark.parametrize("Hkv,S,M", [(8, 1000, 4), (3, 65, 3), (2, 500, 6), (2, 300, 8), (1, 40, 2)])
def test_router_loss_grad_small_column(mq, ref, Hkv, S, M):
    """One expert whose hidden unit the others hardly see (columns of W1 and W2 2^-18, its row of W3 2^-22 of the others): its
    gradients are about 2^-40 of the largest and as exact as theirs."""
    rng = np.random.default_rng(S * 10 + M)
    bits = ((2, 4, 8, 16) * 2)[:M]
    cfg, rcfg = T._cfgs(mq, ref, 1, Hkv, Hkv, 64, 64, bits, 0)
    K, _ = T._rand_kv(rng, 1, Hkv, S)
    W1, W2 = ((rng.standard_normal((128, M)) * 0.1) for _ in range(2))
    W3 = rng.standard_normal((M, M)) * 0.5
    m = M // 2
    W1[:, m] *= 2.0 ** -18; W2[:, m] *= 2.0 ** -18; W3[m] *= 2.0 ** -22
    W1, W2, W3 = (w.astype(np.float16) for w in (W1, W2, W3))
    nll = np.array([2.0], np.float32)
    pm, pe = np.array([1.0 / b for b in bits], np.float32), np.array([16.0 / b for b in bits], np.float32)
    want = ref.router_loss_grad(rcfg, K, 0, S, W1, W2, W3, None, nll, pm, pe, 0.3)
    size = np.abs(want[1]).max(0)
    assert 0 < size[m] <= 2.0 ** -36 * size.max()
    got = [torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in ((3,), (128, M), (128, M), (M, M), (M,))]
    mq.router_loss_grad(cfg, T._dev(K), 0, S, T._dev(W1), T._dev(W2), T._dev(W3), None, T._dev(nll), None, None, 0.3, *got)
    torch.cuda.synchronize()
    _check_columns(("dW1", "dW2"), got[1:3], want[1:3])


@pytest.mark.parametrize("M", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("share,S", [(0.1, 1000), (0.6, 300), (1.0, 65)])
def test_router_loss_grad_some_tokens_tie(mq, ref, M, share, S):
    """Tokens whose two best experts tie take the first of them, as routing does: the other one's penalties differ by a factor."""
    rng = np.random.default_rng(S + M)
    bits = ((2, 16, 4, 8) * 2)[:M]
    cfg, rcfg = T._cfgs(mq, ref, 1, 3, 3, 64, 64, bits, 0)
    K, _ = T._rand_kv(rng, 1, 3, S)
    W1, W2, W3, bias = T._twin_router(rng, M, share, K)
    nll = np.array([2.0], np.float32)
    pm, pe = np.array([1.0 / b for b in bits], np.float32), np.array([16.0 / b for b in bits], np.float32)
    want = ref.router_loss_grad(rcfg, K, 0, S, W1, W2, W3, bias, nll, pm, pe, 0.3)
    got = [torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in ((3,), (128, M), (128, M), (M, M), (M,))]
    mq.router_loss_grad(cfg, T._dev(K), 0, S, T._dev(W1), T._dev(W2), T._dev(W3), T._dev(bias), T._dev(nll), None, None, 0.3, *got)
    torch.cuda.synchronize()
    l = got[0].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(l - want[0]) <= LOSS_TOL * np.abs(want[0]).max()), (l, want[0])
    for g, r in zip(got[1:], want[1:]):
        assert np.abs(g.cpu().numpy() - r).max() <= GRAD_TOL * np.abs(r).max()


@pytest.mark.parametrize("M", [2, 4, 5, 8])
@pytest.mark.parametrize("kind", ["keys", "weights"])
def test_router_loss_grad_subnormal_operands(mq, ref, kind, M):
    """Two experts that tie but for the order of their sums, of subnormal keys or weights: the top-1 index, and with it the
    penalties (2 and 16 bits), is the one of the sums in order."""
    rng = np.random.default_rng(M)
    bits = ((2, 16, 4, 8) * 2)[:M]
    cfg, rcfg = T._cfgs(mq, ref, 1, 2, 2, 64, 64, bits, 0)
    K, W1, W2, W3 = T._subnormal_twins(rng, kind, 1, 2, 500, M)
    nll = np.array([2.0], np.float32)
    pm, pe = np.array([1.0 / b for b in bits], np.float32), np.array([16.0 / b for b in bits], np.float32)
    want = ref.router_loss_grad(rcfg, K, 0, 500, W1, W2, W3, None, nll, pm, pe, 0.3)
    got = [torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in ((3,), (128, M), (128, M), (M, M), (M,))]
    mq.router_loss_grad(cfg, T._dev(K), 0, 500, T._dev(W1), T._dev(W2), T._dev(W3), None, T._dev(nll), None, None, 0.3, *got)
    torch.cuda.synchronize()
    l = got[0].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(l - want[0]) <= LOSS_TOL * np.abs(want[0]).max()), (l, want[0])


@pytest.mark.parametrize("M,S,kind", [(1, 4096, "ties"), (2, 4096, "ties"), (2, 4096, "subnormal"), (2, 4033, "ties"), (2, 4032, "ties")])
def test_router_loss_grad_many_tiles(mq, ref, M, S, kind):
    """One and two experts from two tiles per wavefront on (64 rows of 64 tiles on 256 compute units; 63 tiles are too few): the
    forward pass on the matrix cores, which the smaller calls of these do not take."""
    rng = np.random.default_rng(S + M)
    bits = (2, 16)[:M]
    cfg, rcfg = T._cfgs(mq, ref, 1, 64, 64, 64, 64, bits, 0)
    bias = None
    if kind == "subnormal":
        K, W1, W2, W3 = T._subnormal_twins(rng, "keys", 1, 64, S, M)
    else:
        K, _ = T._rand_kv(rng, 1, 64, S)
        W1, W2, W3, bias = T._twin_router(rng, 2, 0.05, K)
        W1, W2, W3, bias = W1[:, :M].copy(), W2[:, :M].copy(), W3[:M, :M].copy(), bias[:M].copy()
    nll = np.array([2.0], np.float32)
    pm, pe = np.array([1.0 / b for b in bits], np.float32), np.array([16.0 / b for b in bits], np.float32)
    want = ref.router_loss_grad(rcfg, K, 0, S, W1, W2, W3, bias, nll, pm, pe, 0.3)
    got = [torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in ((3,), (128, M), (128, M), (M, M), (M,))]
    mq.router_loss_grad(cfg, T._dev(K), 0, S, T._dev(W1), T._dev(W2), T._dev(W3), None if bias is None else T._dev(bias), T._dev(nll),
                        None, None, 0.3, *got)
    torch.cuda.synchronize()
    l = got[0].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(l - want[0]) <= LOSS_TOL * np.abs(want[0]).max()), (l, want[0])
    if kind != "subnormal":                                       # (whose gradients are of the order of 1e-20)
        for g, r in zip(got[1:], want[1:]):
            assert np.abs(g.cpu().numpy() - r).max() <= GRAD_TOL * max(np.abs(r).max(), 1e-6)
