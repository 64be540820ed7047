"""Prefill path (MFMA grouped GEMM) against the oracle, through the C ABI."""
import numpy as np
import pytest

from oracle import moe_oracle as O
from synth import configs as C

import gpu_support as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_01433_amd as P
    P.lib()
    yield


def _edge(name, seed, d, f, E, K, T, tags, t1=1.0, t2=1.0):
    return C.Workload(name=name, seed=seed, d_model=d, d_ff=f, n_experts=E,
                      top_k=K, n_tokens=T, t1=t1, t2=t2, fixed_tags=tuple(tags))


def run_prefill(L, x16, d, K, residual_h=None):
    T = x16.shape[0]
    xd = torch.from_numpy(np.ascontiguousarray(x16)).cuda()
    idx = torch.empty((T, K), dtype=torch.int32, device="cuda")
    w = torch.empty((T, K), dtype=torch.float32, device="cuda")
    prec = torch.empty((T, K), dtype=torch.int8, device="cuda")
    if residual_h is None:
        y = torch.empty((T, d), dtype=torch.float32, device="cuda")
        L.prefill(xd, y, idx, w, prec)
        torch.cuda.synchronize()
        return y.cpu().numpy(), idx.cpu().numpy(), w.cpu().numpy(), prec.cpu().numpy()
    xn = torch.empty((T, d), dtype=torch.float16, device="cuda")
    L.prefill_residual(xd, residual_h, xn, idx, w, prec)
    torch.cuda.synchronize()
    return xn.cpu().numpy(), idx.cpu().numpy(), w.cpu().numpy(), prec.cpu().numpy()


def _check(wl, tags, x16, sample=None, t1=None, t2=None, residual=False):
    t1 = wl.t1 if t1 is None else t1
    t2 = wl.t2 if t2 is None else t2
    weights = S.device_layer_weights(wl, 0)
    L = S.make_layer(wl, tags, weights, max_tokens=len(x16), t1=t1, t2=t2)
    K, d = wl.top_k, wl.d_model
    if residual:
        h0 = np.asarray(x16, dtype=np.float32) * np.float32(0.25)
        hd = torch.from_numpy(h0).cuda()
        xn, idx, w, prec = run_prefill(L, x16, d, K, residual_h=hd)
        out = hd.cpu().numpy() - h0
    else:
        out, idx, w, prec = run_prefill(L, x16, d, K)
    L.destroy()
    # routing of every token; the fp64 expert FFN on the sampled rows
    wg16 = C.router_weight(wl, 0)
    r_all, flags = S.check_routing(x16, wg16, tags, K, t1, t2, idx, w, prec)
    rows = np.arange(len(x16)) if sample is None else np.asarray(sample)
    r = O.Routing(idx=r_all.idx[rows], w=r_all.w[rows], prec=r_all.prec[rows],
                  logits=r_all.logits[rows])
    y_ref = O.layer_output(x16[rows], S.HostExperts(wl, 0, tags), r)
    err = S.normwise(out[rows], y_ref)
    print(f"{wl.name}: routing exact on {len(x16)} tokens ({len(flags)} flagged near-ties); "
          f"max normwise err {err.max():.3e} over {len(rows)} tokens")
    assert err.max() <= S.TOL
    if residual:
        h_ref = h0[rows].astype(np.float64) + y_ref
        assert S.normwise(xn[rows], O.rmsnorm(h_ref)).max() <= S.TOL
    return idx, prec


def test_prefill_tiny():
    wl = C.TINY
    _check(wl, C.layer_tags(wl, 0), C.hidden_states(wl))


def test_prefill_tiny_many_tokens_all_tags():
    """Groups of about 210 tokens at every width (fp16, int4,
    int2); every tag kind."""
    wl = _edge("prefill_busy", 41, 256, 512, 4, 2, 420,
               [C.TAG_FP16, C.TAG_INT4, C.TAG_INT2, C.TAG_MISS_INT4], t1=0.45, t2=1.0)
    rng = np.random.default_rng(11)
    idx, prec = _check(wl, wl.fixed_tags, rng.standard_normal((420, 256)).astype(np.float16))
    counts = np.bincount(idx.ravel(), minlength=4)
    assert counts[:3].min() > 160, counts


def test_prefill_ragged_shapes():
    wl = _edge("prefill_ragged", 42, 192, 320, 5, 3, 37,
               [C.TAG_FP16, C.TAG_INT4, C.TAG_INT2, C.TAG_MISS_INT4, C.TAG_MISS_INT2],
               t1=0.4, t2=0.8)
    rng = np.random.default_rng(12)
    _check(wl, wl.fixed_tags, rng.standard_normal((37, 192)).astype(np.float16))


def test_prefill_skip_and_residual():
    wl = _edge("prefill_skip", 43, 256, 384, 6, 2, 50, [C.TAG_MISS_INT2] * 6)
    rng = np.random.default_rng(13)
    x = rng.standard_normal((50, 256)).astype(np.float16)
    _check(wl, wl.fixed_tags, x, t1=0.0, t2=0.0, residual=True)
    _check(wl, wl.fixed_tags, x, t1=0.0, t2=1.0)


def test_prefill_max_tokens():
    """The largest step a layer takes (8192 tokens): about 2,000 tokens per
    group, i.e. 8 or 9 token tiles per weight tile, every tag kind; routing
    of all tokens, the output on 512 evenly spread tokens."""
    T = 8192
    wl = _edge("prefill_max", 44, 256, 512, 8, 2, T,
               [C.TAG_FP16, C.TAG_INT4, C.TAG_INT2, C.TAG_MISS_INT4, C.TAG_MISS_INT2,
                C.TAG_FP16, C.TAG_MISS_INT4, C.TAG_INT4], t1=0.3, t2=0.6)
    rng = np.random.default_rng(14)
    x = rng.standard_normal((T, 256)).astype(np.float16)
    idx, prec = _check(wl, wl.fixed_tags, x, sample=np.linspace(0, T - 1, 512).astype(int))
    counts = np.bincount(idx.ravel(), minlength=8)
    assert counts.min() > 160, counts
    # all three outcomes of Eq. 2 occur on the miss-tagged experts
    assert {0, 1, 2} <= set(np.unique(prec).tolist()), np.unique(prec)


def test_prefill_mixtral_layer_t512():
    """One Mixtral-shaped layer of the 512-token prefill workload (4:3:1
    map of layer 0): routing of all 512 tokens, the layer output on 32
    sampled tokens, against the oracle."""
    wl = C.MIXTRAL_PREFILL
    tags = C.layer_tags(wl, 0)
    x = C.hidden_states(wl)
    sample = np.linspace(0, wl.n_tokens - 1, 32).astype(int)
    _check(wl, tags, x, sample=sample)


def test_prefill_matches_decode():
    wl = C.MIXTRAL_T8_SKEW
    tags = C.layer_tags(wl, 0)
    weights = S.device_layer_weights(wl, 0)
    L = S.make_layer(wl, tags, weights)
    x = C.hidden_states(wl)
    y_p, idx_p, _, prec_p = run_prefill(L, x, wl.d_model, wl.top_k)
    y_d, idx_d, _, prec_d = S.run_decode(L, torch.from_numpy(x).cuda(), wl.n_tokens,
                                         wl.d_model, wl.top_k)
    L.destroy()
    assert np.array_equal(idx_p, idx_d) and np.array_equal(prec_p, prec_d)
    assert S.normwise(y_p, y_d).max() <= S.TOL


# One expert, so that its group has exactly T tokens: the edges of the token
# tiles (32 each, up to 256 per block) and of the next block, the number
# of reduction stages from one (d 64) over fewer than the staging rings hold
# to many, and weight rows that fill no tile.  d 1088 with 8192 tokens takes
# the 256-row blocks in both projections, the others the 128-row ones.
@pytest.mark.parametrize("tag", [C.TAG_FP16, C.TAG_INT8, C.TAG_INT4, C.TAG_INT2])
@pytest.mark.parametrize("d,f,T", [(64, 64, 1), (64, 192, 64), (192, 64, 65), (320, 448, 128),
                                   (576, 320, 129), (128, 704, 160), (448, 128, 193),
                                   (256, 576, 32), (192, 448, 33), (704, 320, 96),
                                   (64, 320, 224), (1024, 128, 225), (832, 192, 256), (192, 832, 257), (320, 192, 513),
                                   (1088, 704, 8192)])
def test_prefill_tile_edges(tag, d, f, T):
    wl = _edge(f"prefill_edge_{tag}_{d}_{f}_{T}", 45, d, f, 1, 1, T, [tag])
    x = np.random.default_rng(15).standard_normal((T, d)).astype(np.float16)
    sample = np.unique(np.linspace(0, T - 1, 600).astype(int))
    _check(wl, wl.fixed_tags, x, sample=sample)


# The same in the 256-row blocks of both projections, whose rings differ with
# the number of token tiles in the last block: one expert with 31 full blocks
# and a remainder of 1 to 7 tiles of 32 tokens (the 8 tiles are above).
@pytest.mark.parametrize("tag", [C.TAG_FP16, C.TAG_INT8, C.TAG_INT4, C.TAG_INT2])
@pytest.mark.parametrize("rest", [1, 33, 65, 97, 129, 161, 193])
def test_prefill_large_block_remainders(tag, rest):
    d, f, T = 1088, 704, 31 * 256 + rest
    wl = _edge(f"prefill_rest_{tag}_{rest}", 48, d, f, 1, 1, T, [tag])
    x = np.random.default_rng(18).standard_normal((T, d)).astype(np.float16)
    _check(wl, wl.fixed_tags, x, sample=np.r_[np.linspace(0, T - rest - 1, 40).astype(int),
                                              T - rest:T])


@pytest.mark.parametrize("E,K,T", [(64, 8, 700), (64, 1, 8192), (3, 2, 4000)])
def test_prefill_many_groups(E, K, T):
    """Work lists of up to 128 groups (both copies of every expert), of groups
    that are all small, and of few large ones with remainders."""
    wl = _edge(f"prefill_groups_{E}_{K}_{T}", 46, 128, 192, E, K, T,
               [(C.TAG_MISS_INT4, C.TAG_MISS_INT2, C.TAG_MISS_INT8_INT2)[e % 3] for e in range(E)],
               t1=0.3, t2=0.9)
    x = np.random.default_rng(16).standard_normal((T, 128)).astype(np.float16)
    _check(wl, wl.fixed_tags, x, sample=np.unique(np.linspace(0, T - 1, 500).astype(int)))


@pytest.mark.parametrize("T", [512, 513, 2047, 2048, 2049])
@pytest.mark.parametrize("E,K", [(6, 3), (17, 2)])
def test_prefill_router_block_sizes(E, K, T):
    """Either side of the step sizes from which the router's blocks take 4 and
    16 tokens, with gate rows in registers (E <= 16) and from L2."""
    wl = _edge(f"prefill_router_{E}_{T}", 47, 128, 64, E, K, T,
               [(C.TAG_FP16, C.TAG_MISS_INT4, C.TAG_MISS_INT2)[e % 3] for e in range(E)],
               t1=0.3, t2=0.8)
    x = np.random.default_rng(17).standard_normal((T, 128)).astype(np.float16)
    _check(wl, wl.fixed_tags, x, sample=np.unique(np.linspace(0, T - 1, 400).astype(int)))


@pytest.mark.parametrize("T,call", [(64, "prefill"), (2048, "prefill"), (64, "decode_step")])
def test_swiglu_is_exact_to_fp32(T, call):
    """One expert with diagonal weights: a[r] = x[r] w[r], b[r] = 2^k[r] x[r]
    and y = h, so that every SwiGLU value shows.  Gates of -8 to -25, where
    e^-a magnifies an error of its exponent the most.  In fp32 the exponential
    is good to 1.5 ulp (3 x 2^-24 of its value), and the sum, the quotient and
    the product are rounded once each (2^-24): at most 6 x 2^-24 from 64
    bits.  So h is the fp16 number next to the exact value, unless that lies
    within that distance of the middle between two of them."""
    import paper_2411_01433_amd as P
    d = 512
    rng = np.random.default_rng(70 + T)
    w = rng.uniform(1, 2, d).astype(np.float16)
    a = -rng.uniform(8, 25, (T, d))
    a[:, 1::2] = np.maximum(a[:, 1::2], -18)
    x = (a / w).astype(np.float16)
    k = np.where(np.arange(d) % 2 == 0, 15, 10)                # h is a normal fp16 number
    diag = lambda v: torch.diag(torch.from_numpy(v.astype(np.float16)).cuda()).contiguous()
    wg = torch.ones((1, d), dtype=torch.float16, device="cuda")
    w1, w3, w2 = diag(w), diag(2.0 ** k), diag(np.ones(d))
    L = P.MoeLayer(d, d, 1, 1, T, wg, [w1], [w3], [w2])
    y = torch.empty((T, d), dtype=torch.float32, device="cuda")
    getattr(L, call)(torch.from_numpy(x).cuda(), y)
    torch.cuda.synchronize()
    L.destroy()
    a = x.astype(np.float64) * w.astype(np.float64)
    exact = a / (1.0 + np.exp(-a)) * (x.astype(np.float64) * 2.0 ** k)
    ulp = 2.0 ** (np.floor(np.log2(exact)) - 10)
    assert exact.min() > 2.0 ** -14 and exact.max() < 65504
    off = np.abs(y.cpu().numpy() - exact) - ulp / 2              # beyond the nearest fp16 number
    bad = off > 6 * 2.0 ** -24 * exact
    print(f"{bad.sum()} of {bad.size} values further off; the worst by {(off / exact).max():.2e}")
    assert not bad.any()
