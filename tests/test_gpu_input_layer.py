"""GPU parity of the sparse input layer (section 2.2) against oracle.input_layer,
through the C ABI.  Inputs: the synth generators' (index, value) pairs as the
K-sparse inputs x and their H as dL/dA."""
import functools

import numpy as np
import pytest

from oracle import input_layer
from synth import Workload, WorkloadConfig, get_config

from parity_util import rel

pytestmark = pytest.mark.gpu


def _layer(W):
    import torch

    import paper_1412_7091_amd as lst

    return lst.SparseInputLayer(torch.from_numpy(W).cuda())


def _check_steps(cfg, steps, lr):
    import torch

    wl = Workload(cfg)
    W = wl.init_V()
    layer = _layer(W)
    W_ref = W.astype(np.float64)
    for s in range(steps):
        G, idx, val = wl.batch(s)            # G plays dL/dA (m x d)
        i_t, v_t = torch.from_numpy(idx).cuda(), torch.from_numpy(val).cuda()
        A = layer.forward(i_t, v_t).cpu().numpy()
        A_ref = input_layer.forward(W_ref, idx, val)
        # each row is a sum of at most K products: fp32 rounding only
        assert rel(A, A_ref) < 1e-6, (s, rel(A, A_ref))
        W_prev = layer.get_W().cpu().numpy()
        layer.update(i_t, v_t, torch.from_numpy(G).cuda(), lr)
        assert layer.sync() == 0
        W_new = layer.get_W().cpu().numpy()
        W_ref = input_layer.update(W_ref, idx, val, G, lr)
        touched = np.unique(idx[idx >= 0])
        mask = np.ones(W.shape[0], dtype=bool)
        mask[touched] = False
        assert np.array_equal(W_new[mask], W_prev[mask]), "a row no input refers to changed"
        assert rel(W_new[touched], W_ref[touched]) < 1e-6
    layer.close()


@pytest.mark.parametrize("d", [40, 37])
def test_input_layer_small_with_repeats(gpu_lib, d):
    cfg = WorkloadConfig(name="inp", D=300, d=d, m=24, K=6, idx_dist="uniform", distinct=False,
                         val_dist="normal", pad_frac=0.2, dup_frac=0.3, entropy=4000 + d)
    _check_steps(cfg, 4, 0.05)


@pytest.mark.parametrize("d", [300, 37])
def test_input_layer_long_lists(gpu_lib, d):
    """K = 300 > 16: the forward pass splits each list into quarters over four waves."""
    cfg = WorkloadConfig(name="inpl", D=3000, d=d, m=12, K=300, idx_dist="uniform",
                         distinct=False, val_dist="normal", pad_frac=0.1, dup_frac=0.2,
                         entropy=4400 + d)
    _check_steps(cfg, 2, 0.01)


def test_input_layer_zipf_shared_rows(gpu_lib):
    cfg = WorkloadConfig(name="inpz", D=5000, d=64, m=128, K=8, idx_dist="zipf", zipf_s=1.1,
                         distinct=True, val_dist="one", entropy=4100)
    _check_steps(cfg, 3, 0.01)


def test_input_layer_full_size(gpu_lib):
    """D_in = 200 000, d = 500, m = 128 examples with 10 input pairs each."""
    cfg = get_config("c2")
    _check_steps(cfg, 2, 1e-3)


def test_input_layer_max_slots_zipf(gpu_lib):
    """m K = 65 536 slots (the largest call), Zipf 1.1 inputs: rows held by thousands of
    slots next to rows held by one; two calls, so the row table must be left empty."""
    cfg = WorkloadConfig(name="inpmax", D=20000, d=40, m=512, K=128, idx_dist="zipf",
                         zipf_s=1.1, distinct=False, val_dist="normal", entropy=4300)
    _check_steps(cfg, 2, 1e-3)


def test_input_layer_bad_index_leaves_W(gpu_lib):
    import torch

    import paper_1412_7091_amd as lst

    cfg = WorkloadConfig(name="inpb", D=500, d=16, m=8, K=3, entropy=4200)
    wl = Workload(cfg)
    W = wl.init_V()
    layer = _layer(W)
    G, idx, val = wl.batch(0)
    idx[3, 1] = cfg.D                          # out of range
    layer.update(torch.from_numpy(idx).cuda(), torch.from_numpy(val).cuda(),
                 torch.from_numpy(G).cuda(), 0.1)
    assert layer.sync() == lst.LST_EINDEX
    assert np.array_equal(layer.get_W().cpu().numpy(), W)
    # the rejected call still emptied its row table: the next call is exact
    G1, idx1, val1 = wl.batch(1)
    layer.update(torch.from_numpy(idx1).cuda(), torch.from_numpy(val1).cuda(),
                 torch.from_numpy(G1).cuda(), 0.1)
    assert layer.sync() == 0
    W_ref = input_layer.update(W.astype(np.float64), idx1, val1, G1, 0.1)
    assert rel(layer.get_W().cpu().numpy(), W_ref) < 1e-6
    layer.close()


@pytest.mark.parametrize("kw", [
    dict(m=1, K=1, d=5, D=3),                                  # the smallest call
    dict(m=64, K=4, d=64, D=40),                               # 256 slots: the short small form
    dict(m=257, K=1, d=30, D=100),
    dict(m=128, K=16, d=258, D=60),                            # 2048: one launch, hot rows
    dict(m=683, K=3, d=500, D=1000),                           # 2049: the grouped form
    dict(m=1, K=2048, d=513, D=7),                             # every row hot
    dict(m=1, K=2100, d=1030, D=9),
    dict(m=61, K=63, d=64, D=5000, idx_dist="zipf", zipf_s=1.1),
    dict(m=1024, K=64, d=36, D=50),                            # every row hot, all 64 blocks
    dict(m=4096, K=16, d=20, D=30000, idx_dist="zipf", zipf_s=1.0),
    dict(m=65535, K=1, d=12, D=1),                             # one row, every slot
    dict(m=16384, K=1, d=33, D=3000),                          # 64 sorted blocks of 256
    dict(m=1024, K=16, d=3, D=50),                             # and every row hot in all of them
    dict(m=16385, K=1, d=66, D=20000),                         # blocks of 1024
    dict(m=9, K=300, d=257, D=500),                            # lists of more than 64 a quarter
    dict(m=40, K=61, d=6, D=400),
])
def test_input_layer_forms_and_edges(gpu_lib, kw):
    """The update's forms at their edges (256, 2048, 16 384 slots; 64 slots a row; 256 and 1024
    slots a sorted block), with pads and repeats; the forward pass at K = 16 and beyond.  With u =
    2^-24, an element is off by at most u times its longest chain of roundings times the sum of
    its terms' magnitudes: the product and up to 64 additions in a group, 4 groups in a part,
    n / 256 parts, and the subtraction from W (forward: K additions, or a quarter of them and
    3).  For terms of random sign the roundings of a chain of k add up as sqrt(k) times u times
    the partial sums, which are about as large as the result: 1.1e-6 of it at n = 65 536
    (k = 326), for which the norm of the change has 1e-5."""
    cfg = WorkloadConfig(name="inpf", distinct=False, val_dist="normal", pad_frac=0.15,
                         dup_frac=0.2, entropy=4500 + kw["m"] + 7 * kw["K"] + kw["d"],
                         **{"idx_dist": "uniform", **kw})
    import torch

    wl = Workload(cfg)
    W = wl.init_V()
    layer = _layer(W)
    lr = float(np.float32(0.01))
    for s in range(2):
        G, idx, val = wl.batch(s)
        i_t, v_t = torch.from_numpy(idx).cuda(), torch.from_numpy(val).cuda()
        A = layer.forward(i_t, v_t).cpu().numpy().astype(np.float64)
        W_prev = layer.get_W().cpu().numpy()
        layer.update(i_t, v_t, torch.from_numpy(G).cuda(), lr)
        assert layer.sync() == 0
        W_new = layer.get_W().cpu().numpy()
        A_ref, dW = np.zeros((cfg.m, cfg.d)), np.zeros((cfg.D, cfg.d))
        A_abs, dW_abs = A_ref.copy(), dW.copy()
        rows, cols = np.nonzero(idx >= 0)
        at = idx[rows, cols]
        v64 = val[rows, cols].astype(np.float64)
        np.add.at(A_ref, rows, v64[:, None] * W_prev[at].astype(np.float64))
        np.add.at(A_abs, rows, np.abs(v64[:, None] * W_prev[at]))
        np.add.at(dW, at, v64[:, None] * G[rows].astype(np.float64))
        np.add.at(dW_abs, at, np.abs(v64[:, None] * G[rows]))
        assert rel(A, A_ref) < 1e-6 + 2.0 ** -24 * np.sqrt(cfg.K), rel(A, A_ref)
        chain = cfg.K if cfg.K <= 16 else -(-cfg.K // 4) + 3
        assert np.all(np.abs(A - A_ref) <= 2.0 ** -24 * (chain + 1) * A_abs)
        W_ref = W_prev.astype(np.float64) - lr * dW
        n = np.bincount(at, minlength=cfg.D)[:, None]
        chain = np.minimum(n, 64) + np.minimum(-(-n // 64), 4) + -(-n // 256)
        # (1.01: the second-order terms)
        bound = 1.01 * 2.0 ** -24 * ((chain + 2) * lr * dW_abs + np.abs(W_ref))
        assert np.all(np.abs(W_new - W_ref) <= bound)
        touched = np.unique(at)
        rest = np.setdiff1d(np.arange(cfg.D), touched)
        assert np.array_equal(W_new[rest], W_prev[rest])
        e = rel(W_new[touched] - W_prev[touched].astype(np.float64),
                W_ref[touched] - W_prev[touched].astype(np.float64))
        scale = np.abs(W_prev[touched]).max() / max(np.abs(lr * dW[touched]).max(), 1e-30)
        print(f"{kw}: dW {e:.1e}", flush=True)
        # the change itself, to the rounding of its sum and of W
        assert e < 1e-5 + 2.0 ** -23 * scale, e
        assert rel(W_new[touched], W_ref[touched]) < 1e-6
    layer.close()


@pytest.mark.parametrize("m,K", [(16, 8), (100, 30)])
def test_input_layer_bad_index_both_forms(gpu_lib, m, K):
    """A bad index in an update of one launch (128 slots) and of the grouped form (3000):
    reported, W unchanged, the next call exact; the forward pass leaves its pair out."""
    import torch

    import paper_1412_7091_amd as lst

    cfg = WorkloadConfig(name="inpbb", D=400, d=24, m=m, K=K, distinct=False, entropy=4600 + m)
    wl = Workload(cfg)
    W = wl.init_V()
    layer = _layer(W)
    G, idx, val = wl.batch(0)
    bad = idx.copy()
    bad[m // 2, 1], bad[m - 1, K - 1] = cfg.D, -2
    t = [torch.from_numpy(x).cuda() for x in (bad, val, G)]
    layer.update(*t, 0.1)
    assert layer.sync() == lst.LST_EINDEX
    assert np.array_equal(layer.get_W().cpu().numpy(), W)
    A = layer.forward(t[0], t[1]).cpu().numpy()
    assert layer.sync() == lst.LST_EINDEX
    good = np.where((bad >= 0) & (bad < cfg.D), bad, -1)
    assert rel(A, input_layer.forward(W.astype(np.float64), good, val)) < 1e-6
    layer.update(torch.from_numpy(idx).cuda(), t[1], t[2], 0.1)
    assert layer.sync() == 0
    W_ref = input_layer.update(W.astype(np.float64), idx, val, G, 0.1)
    assert rel(layer.get_W().cpu().numpy(), W_ref) < 1e-6
    layer.close()


def _documented_update(W, idx, val, G, lr):
    """lst_input_update's sums in float32 in the order its header states: pairs in (example,
    pair) order; from 64 pairs a row on, groups of 64, four groups to a part, then the parts."""
    W = W.copy()
    ex, k = np.nonzero(idx >= 0)
    rows = idx[ex, k]
    for r in np.unique(rows):
        at = rows == r
        terms = val[ex[at], k[at]][:, None] * G[ex[at]]
        add = lambda xs: functools.reduce(np.add, xs, np.zeros(W.shape[1], np.float32))
        if len(terms) >= 64:
            groups = [add(terms[o:o + 64]) for o in range(0, len(terms), 64)]
            terms = [add(groups[o:o + 4]) for o in range(0, len(groups), 4)]
        W[r] -= np.float32(lr) * add(terms)
    return W


@pytest.mark.parametrize("d", [37, 64, 516])
@pytest.mark.parametrize("pairs", [(1, 63, 64, 65, 255), (256, 257, 320), (321, 512, 513),
                                   (1700,)])
def test_input_layer_order_of_sums(gpu_lib, pairs, d):
    """A row's pairs are added in the documented order, in the one-launch form (m K = 2048) and,
    with one more unused slot an example, in the grouped one (2176): both equal the same sums in
    float32 bit for bit.  Values and rate are powers of two, so that products are exact and a
    fused multiply-add rounds as the addition does."""
    import torch

    rng = np.random.default_rng(sum(pairs) + d)
    m, K = 128, 16
    idx = np.full(m * K, -1, np.int32)
    slots = rng.permutation(m * K)[:sum(pairs)]
    idx[slots] = np.repeat(np.arange(len(pairs)), pairs)
    idx = idx.reshape(m, K)
    val = np.exp2(rng.integers(-2, 3, (m, K))).astype(np.float32)
    G = rng.standard_normal((m, d)).astype(np.float32)
    W = rng.standard_normal((len(pairs) + 2, d)).astype(np.float32)
    want = _documented_update(W, idx, val, G, 0.125)
    for pad in (0, 1):
        layer = _layer(W)
        i_t = torch.from_numpy(np.pad(idx, ((0, 0), (0, pad)), constant_values=-1)).cuda()
        v_t = torch.from_numpy(np.pad(val, ((0, 0), (0, pad)))).cuda()
        layer.update(i_t, v_t, torch.from_numpy(G).cuda(), 0.125)
        assert layer.sync() == 0
        got = layer.get_W().cpu().numpy()
        assert np.array_equal(got, want), (pad, np.abs(got - want).max(axis=1))
        layer.close()


@pytest.mark.parametrize("pairs,d", [
    ((32768,), 512),                                           # 128 parts of 8 chunks: narrow
    ((32769,), 512),                                           # 129: 512 columns a block
    ((24321,), 700),                                           # two of them
    ((53000,), 301),                                           # rows not aligned
    ((30000, 20000, 300, 256, 64, 63, 1), 330),                # rows of one part and of many
])
def test_input_layer_order_of_long_sums(gpu_lib, pairs, d):
    """The same for the parts of hot rows on either side of the line (1024 parts times 64-column
    chunks) from which a block takes 512 columns of a part."""
    import torch

    rng = np.random.default_rng(sum(pairs) + d)
    m, K = 1024, 64
    idx = np.full(m * K, -1, np.int32)
    idx[rng.permutation(m * K)[:sum(pairs)]] = np.repeat(np.arange(len(pairs)), pairs)
    idx = idx.reshape(m, K)
    val = np.exp2(rng.integers(-2, 3, (m, K))).astype(np.float32)
    G = rng.standard_normal((m, d)).astype(np.float32)
    W = rng.standard_normal((len(pairs) + 1, d)).astype(np.float32)
    layer = _layer(W)
    layer.update(*(torch.from_numpy(x).cuda() for x in (idx, val, G)), 0.125)
    assert layer.sync() == 0
    got = layer.get_W().cpu().numpy()
    layer.close()
    want = _documented_update(W, idx, val, G, 0.125)
    assert np.array_equal(got, want), np.abs(got - want).max(axis=1)


@pytest.mark.parametrize("kw", [
    dict(m=1024, K=64, d=36, D=50),                            # every row of several parts
    dict(m=4096, K=16, d=20, D=30000, idx_dist="zipf", zipf_s=1.0),
    dict(m=61, K=63, d=64, D=5000, idx_dist="zipf", zipf_s=1.1),
])
def test_input_layer_grouped_update_repeats(gpu_lib, kw):
    """The grouped update lists its rows and parts in the order that blocks arrive; the sums do
    not depend on it: layers of the same W give the same bits, call after call."""
    import torch

    wl = Workload(WorkloadConfig(name="inpr", distinct=False, val_dist="normal", pad_frac=0.1,
                                 dup_frac=0.2, entropy=4700 + kw["m"],
                                 **{"idx_dist": "uniform", **kw}))
    W = wl.init_V()
    layers = [_layer(W) for _ in range(3)]
    for s in range(3):
        G, idx, val = (torch.from_numpy(x).cuda() for x in wl.batch(s))
        got = []
        for layer in layers:
            layer.update(idx, val, G, 0.01)
            assert layer.sync() == 0
            got.append(layer.get_W().cpu().numpy())
        assert not np.array_equal(got[0], W)
        assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
        W = got[0]
    for layer in layers:
        layer.close()


@pytest.mark.parametrize("m,K,d", [(3, 5, 4), (100, 12, 260), (130, 20, 512), (700, 4, 36)])
def test_input_layer_unaligned_buffers(gpu_lib, m, K, d):
    """Activations and gradients that start at a 4-byte address take the same sums in the same
    order as aligned ones: equal bits."""
    import torch

    rng = np.random.default_rng(m + K + d)
    W = rng.standard_normal((90, d)).astype(np.float32)
    idx = torch.from_numpy(rng.integers(-1, 90, (m, K)).astype(np.int32)).cuda()
    val = torch.from_numpy(rng.standard_normal((m, K)).astype(np.float32)).cuda()
    G = torch.from_numpy(rng.standard_normal((m, d)).astype(np.float32)).cuda()
    results = []
    for off in (0, 1):
        layer = _layer(W)
        G_o, A = (torch.empty(m * d + 4, device="cuda")[off:off + m * d].view(m, d)
                  for _ in range(2))
        G_o.copy_(G)
        layer.update(idx, val, G_o, 0.03)
        layer.forward(idx, val, out=A)
        assert layer.sync() == 0
        results.append((layer.get_W().cpu().numpy(), A.cpu().numpy()))
        layer.close()
    for a, b in zip(*results):
        assert np.array_equal(a, b)
