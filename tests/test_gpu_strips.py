"""How launches go over the arena: strips of 256 elements, groups of eight,
sparse chunk tables, and workers spread over the waves of a work-group.

Sizes at the edges of a strip (256), a bound word (1024), a strip group (2048)
and a chunk (16384); chunk tables whose groups mostly hold nothing (many
tensors far shorter than a chunk; one, two and three levels of the search over
64 chunks each); worker counts up to one, on and past a work-group's 16 waves.
Every value is compared bit for bit: the kernels and the oracle's fp32 mode
round every written operation alike.  Mid-size problems, past the caches and
past small launches, are too much for the oracle: there the fused rounds of all
workers are compared with per-worker split calls, which go over the strips in
other orders.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2411_17866_amd import arena as A
from paper_2411_17866_amd import dsm

pytestmark = pytest.mark.gpu

EDGES = [1, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049]
SPARSE_64 = (EDGES * 7)[:64]                        # one level of the search
SPARSE_130 = EDGES * 12 + [40003, 16384, 0] + EDGES     # two, and full chunks among them
SPARSE_4100 = ([3, 1, 260] * 1400)[:4100]           # three
DENSE = [16384, 32769, 14337, 5, 16383]
LAYOUTS = [dsm.DSM_REPLICAS_CONTIGUOUS, dsm.DSM_REPLICAS_BLOCKED, dsm.DSM_REPLICAS_STATE_BLOCKED]
LOCAL = {dsm.DSM_BASE_ADAMW: dict(lr=1e-3, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1),
         dsm.DSM_BASE_SGD_MOMENTUM: dict(lr=0.05, beta1=0.9)}
GLOB = dict(eta=0.8, beta1=0.95, beta2=0.98, lam=0.1)


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().copy()


def tensors(ar, flat):
    h = host(flat)
    return [h[o:o + k].copy() for o, k in zip(ar.offsets, ar.numel)]


def same_bits(got, want, what):
    for p, (a, b) in enumerate(zip(got, want)):
        assert np.array_equal(a.view(np.uint32), np.asarray(b, np.float32).view(np.uint32)), (what, p)


def padding(ar, flat):
    keep = np.ones(flat.numel(), dtype=bool)
    for o, k in zip(ar.offsets, ar.numel):
        keep[o:o + k] = False
    return host(flat)[keep]


@pytest.mark.parametrize("numel,n,base,mode,layout,fused", [
    (SPARSE_130, 1, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_DET, 0, True),
    (SPARSE_130, 3, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_RAND_FLIP, 0, True),
    (SPARSE_130, 5, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_RAND_ZERO, 1, True),
    (SPARSE_130, 16, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_RAND_FLIP, 2, True),
    (SPARSE_130, 17, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_RAND_FLIP, 2, True),
    (SPARSE_130, 2, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_RAND_FLIP, 1, False),
    (SPARSE_64, 6, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_RAND_ZERO, 0, False),
    (SPARSE_4100, 2, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_RAND_FLIP, 2, True),
    (DENSE, 4, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_RAND_ZERO, 1, True),
    (DENSE, 5, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_RAND_FLIP, 0, True),
    (DENSE, 15, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_RAND_FLIP, 2, True),
    (DENSE, 9, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_RAND_ZERO, 0, True),
    (DENSE, 17, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_DET, 0, True),
    (DENSE, 33, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_RAND_FLIP, 1, True),
    (DENSE, 9, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_DET, 1, True),
    (DENSE, 20, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_DET, 2, True),
    (DENSE, 64, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_RAND_ZERO, 2, True),
    (DENSE, 7, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_RAND_FLIP, 2, False),
])
def test_rounds_match_oracle(numel, n, base, mode, layout, fused):
    """Three rounds of H = 2 against the oracle's, free-running: from fresh
    replicas, from stale ones (fused: the lazy broadcast), and with a bound
    that shrinks from round to round."""
    H, local = 2, LOCAL[base]
    decay = [p % 3 != 1 for p in range(len(numel))]
    ar = A.Arenas(numel, n, H, base, decay=decay, replica_layout=LAYOUTS[layout])
    gen = torch.Generator(device="cuda").manual_seed(5)
    ar.x.normal_(0.0, 0.02, generator=gen)
    ar.init()
    st = O.init_state(tensors(ar, ar.x), n, "adamw" if base == dsm.DSM_BASE_ADAMW else "sgd")
    pad = padding(ar, ar.x)
    for t in range(3):
        grads = {}
        for k in range(H):
            ar.write_workers("g_rep", torch.empty(n, ar.arena_elems, device="cuda").normal_(
                0.0, 0.01 * 0.1 ** t, generator=gen))
            for i in range(n):
                grads[(i, k)] = tensors(ar, ar.worker("g_rep", i))
            s = t * H + k + 1
            if fused and k == H - 1:
                dsm.dsm_round_end(ar.ctx, s, local, t, gamma=local["lr"], mode=mode, seed=9,
                                  broadcast=False, **GLOB)
            else:
                dsm.dsm_local_step(ar.ctx, -1, s, **local)
        if not fused:
            dsm.dsm_global_step(ar.ctx, t, gamma=local["lr"], mode=mode, seed=9, broadcast=True,
                                **GLOB)
        res = O.communication_round(st, lambda i, k: grads[(i, k)], t, H=H, local=local,
                                    glob=dict(GLOB, mode=mode, seed=9), decay=decay, prec="fp32")
        same_bits(tensors(ar, ar.x), st["x"], f"x, round {t}")
        same_bits(tensors(ar, ar.m), st["m"], f"m, round {t}")
        if mode != dsm.DSM_SIGN_DET:
            B = dsm.dsm_read_bounds(ar.ctx, len(numel))
            want = [np.abs(u).max() if u.size else 0.0 for u in res["u"]]
            assert np.array_equal(B.view(np.uint32), np.asarray(want, np.float32).view(np.uint32))
        for i in range(n):
            if not fused:
                same_bits(tensors(ar, ar.replica(i)), st["x"], f"replica {i}, round {t}")
    assert np.array_equal(padding(ar, ar.x).view(np.uint32), pad.view(np.uint32))
    dsm.dsm_sync(ar.ctx)
    for i in range(n):
        same_bits(tensors(ar, ar.replica(i)), st["x"], f"replica {i} after sync")
    ar.destroy()


@pytest.mark.parametrize("layout", LAYOUTS)
def test_large_randomized_round_end_equals_split(layout):
    """A round end long enough to raise its bound words by atomic maxima (16 x
    8.5M elements) against the split calls on the same inputs."""
    numel, n, base = [8_500_001, 3, 20_001], 16, dsm.DSM_BASE_SGD_MOMENTUM
    got = []
    for fused in (False, True):
        ar = A.Arenas(numel, n, 1, base, replica_layout=layout)
        gen = torch.Generator(device="cuda").manual_seed(6)
        ar.x.normal_(0.0, 0.02, generator=gen)
        ar.init()
        for t in range(2):
            for i in range(n):
                ar.g_rep[i].normal_(0.0, 0.01 * 0.1 ** t, generator=gen)
            if fused:
                dsm.dsm_round_end(ar.ctx, t + 1, LOCAL[base], t, gamma=0.05, seed=9,
                                  mode=dsm.DSM_SIGN_RAND_FLIP, broadcast=True, **GLOB)
            else:
                dsm.dsm_local_step(ar.ctx, -1, t + 1, **LOCAL[base])
                dsm.dsm_global_step(ar.ctx, t, gamma=0.05, seed=9, mode=dsm.DSM_SIGN_RAND_FLIP,
                                    broadcast=True, **GLOB)
        got.append((tensors(ar, ar.x), tensors(ar, ar.m), tensors(ar, ar.replica(n - 1)),
                    [dsm.dsm_read_bounds(ar.ctx, len(numel))]))
        ar.destroy()
        del ar
    for name, a, b in zip(("x", "m", "replica", "bounds"), *got):
        same_bits(b, a, name)


SPARSE_MID = [(k * 7919) % 9_973 + 1 for k in range(400)] + [1_000_003]    # 3M elements
SPARSE_LARGE = [(k * 2741) % 4095 + 2 for k in range(16_000)]              # 33M
MANY_CHUNKS = [40] * 17_000   # with 64 workers more strips than a grid row holds
DENSE_MID = [20_000_003, 5, 16_385]     # strip groups: 9 whole turns of 1024 and a part


@pytest.mark.parametrize("numel,n,base,mode,layout", [
    (SPARSE_MID, 2, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_RAND_FLIP, 2),
    (SPARSE_MID, 6, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_RAND_ZERO, 1),
    (SPARSE_LARGE, 3, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_DET, 0),
    (SPARSE_LARGE, 3, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_RAND_FLIP, 2),
    (MANY_CHUNKS, 64, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_DET, 0),
    (DENSE_MID, 6, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_DET, 0),
    (DENSE_MID, 3, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_RAND_ZERO, 1),
    (DENSE_MID, 2, dsm.DSM_BASE_SGD_MOMENTUM, dsm.DSM_SIGN_RAND_FLIP, 0),
    ([2_000_003, 5, 16_385], 10, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_RAND_FLIP, 2),
    ([1_500_007, 16_384], 10, dsm.DSM_BASE_ADAMW, dsm.DSM_SIGN_RAND_ZERO, 0),
])
def test_mid_size_rounds_equal_per_worker_split_calls(numel, n, base, mode, layout):
    """Two lazy rounds of H = 2 by all-worker local steps and fused round ends
    against the same rounds by one local step call per worker and global steps
    with broadcast."""
    buffers = 4 if base == dsm.DSM_BASE_ADAMW else 3
    assert 4 * sum(numel) * (2 + buffers * n) > 96 << 20    # nontemporal kernels
    H, local, got = 2, LOCAL[base], []
    for fused in (True, False):
        ar = A.Arenas(numel, n, H, base, replica_layout=LAYOUTS[layout])
        gen = torch.Generator(device="cuda").manual_seed(8)
        ar.x.normal_(0.0, 0.02, generator=gen)
        ar.init()
        bounds = []
        for t in range(2):
            for k in range(H):
                s = t * H + k + 1
                for i in range(n):
                    ar.g_rep[i].normal_(0.0, 0.01 * 0.1 ** t, generator=gen)
                if fused and k == H - 1:
                    dsm.dsm_round_end(ar.ctx, s, local, t, gamma=local["lr"], mode=mode, seed=9,
                                      broadcast=False, **GLOB)
                elif fused:
                    dsm.dsm_local_step(ar.ctx, -1, s, **local)
                else:
                    for i in range(n):
                        dsm.dsm_local_step(ar.ctx, i, s, **local)
            if not fused:
                dsm.dsm_global_step(ar.ctx, t, gamma=local["lr"], mode=mode, seed=9,
                                    broadcast=True, **GLOB)
            if mode != dsm.DSM_SIGN_DET:
                bounds.append(dsm.dsm_read_bounds(ar.ctx, len(numel)))
        dsm.dsm_sync(ar.ctx)
        out = {"x": ar.x, "m": ar.m}
        for name in ("s1_rep", "s2_rep", "x_rep"):
            if getattr(ar, name) is not None:
                out.update({f"{name} {i}": ar.worker(name, i) for i in range(n)})
        got.append(({k: v.view(torch.int32).clone() for k, v in out.items()}, bounds))
        ar.destroy()
        del ar, out
    (a, bounds_a), (b, bounds_b) = got
    for name in a:
        assert torch.equal(a[name], b[name]), name
    for x, y in zip(bounds_a, bounds_b):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
