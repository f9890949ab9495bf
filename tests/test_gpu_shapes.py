"""GPU parity at the edges of the kernels' shape ranges (needs an MI355X):
windows that are no multiple of a row tile, lengths around tile, chunk and
segment boundaries, against the fp64 oracle as in test_gpu_parity."""
import pytest

import test_gpu_parity as TP
from oracle import ref
from paper_2606_14782_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ref.set_threads(16)


def _wl(layers, hq, hkv, d, window, pool, dtype, lens, budgets, seed=31):
    return inputs.Workload("shapes", layers, hq, hkv, d, window, pool, dtype, tuple(lens), tuple(budgets),
                           tuple((0, 0) for _ in lens), 0, seed)


@pytest.mark.parametrize("hq,hkv,d,window,lens", [
    (14, 2, 64, 16, (33, 511, 513, 1025)),     # seven 16-query heads: rows end inside a row tile
    (6, 2, 128, 31, (64, 543, 2048)),          # the last query of a head inside a run of four rows
    (6, 2, 64, 33, (2049, 65)),                # a window one row past a tile, keys one past a segment
    (4, 4, 128, 1, (32, 512, 2080)),           # one-row windows: every row a last query
])
def test_window_rows(hq, hkv, d, window, lens):
    """Windows other than 32 queries: the causal edge and the last-query rows
    fall inside row tiles and inside a lane's runs of four rows."""
    wl = _wl(3, hq, hkv, d, window, 5, "bf16", lens, [max(1, n // 8) for n in lens])
    TP.run_case(f"window-{window}", wl, supplied_lse=True)


@pytest.mark.parametrize("hq,hkv,d,window,dtype,lens", [
    (4, 4, 64, 8, "fp32", (512, 130)),           # one row tile: waves without a tile
    (8, 1, 128, 32, "fp32", (700, 4099)),        # 256 rows of fp32: the streaming passes either way
    (4, 1, 128, 32, "fp32", (700, 4099)),        # 128 rows of fp32 d 128: the most fp32 takes there
    (8, 1, 128, 32, "bf16", (700, 4099)),        # 256 rows of bf16 d 128: the most rows
    (6, 2, 128, 8, "fp32", (1030, 70)),          # one row tile, keys spread over the row groups
    (28, 4, 128, 32, "bf16", (513, 2049, 97)),   # seven row tiles over the row groups
    (6, 2, 128, 16, "bf16", (8191, 33)),         # two row tiles, two chunks per workgroup
    (5, 1, 64, 20, "bf16", (6145,)),             # rows that end inside the last tile
    (2, 2, 64, 32, "fp32", (1025, 64, 3000)),
])
@pytest.mark.parametrize("wide", [True, False])
def test_small_grids(hq, hkv, d, window, dtype, lens, wide, monkeypatch):
    """Grids that do not fill the GPU: the wide passes (one launch per layer in
    the prompt call) against the oracle, the prompt call against the per-layer
    calls bit for bit, and the same shapes on the passes of larger grids
    (BACON_WIDE=0)."""
    import torch
    import parity as P
    from paper_2606_14782_amd import bacon
    if not wide:
        monkeypatch.setenv("BACON_WIDE", "0")
    wl = _wl(7, hq, hkv, d, window, 7, dtype, lens, [max(1, n // 10) for n in lens])
    TP.run_case(f"small-grid wide={wide}", wl, split=False, supplied_lse=True)
    batch = bacon.BatchLayout(wl.cu_seqlens, wl.budgets_arr)
    xs = [inputs.layer_inputs(wl, l) for l in range(wl.num_layers)]
    qs, ks, vs = ([P.to_dev(x[n], wl) for x in xs] for n in ("q_win", "k", "v"))
    a, b = P.make_ctx(wl), P.make_ctx(wl)
    for ctx in (a, b):
        ctx.bacon_profile_enable(True)
    a.bacon_begin_prompt(batch)
    want = [a.bacon_compress_layer(l, batch, qs[l], ks[l], vs[l]) for l in range(wl.num_layers)]
    b.bacon_begin_prompt(batch)
    got = b.bacon_compress_prompt(0, batch, qs, ks, vs)
    torch.cuda.synchronize()
    for l in range(wl.num_layers):
        for x, y in zip(got[l], want[l]):
            assert torch.equal(x, y), f"layer {l}"
    # the launches are those of the passes that the case is for
    wide = wide and not (dtype == "fp32" and hq // hkv * window > 128)
    assert ("window_score_calib_wide" in a.bacon_profile_read()) == wide
    assert ("layer_stages" in b.bacon_profile_read()) == wide


@pytest.mark.parametrize("adaptive", [True, False])
@pytest.mark.parametrize("wide", [True, False])
@pytest.mark.parametrize("lse", [False, True])
def test_prompt_longer_than_its_schedule(adaptive, wide, lse, monkeypatch):
    """More layers than the prompt call keeps in flight, so that every buffer's
    copies come round, with budgets that change every layer (per sequence
    under the adaptive allocation, else per head): equal to the per-layer
    calls bit for bit."""
    import numpy as np
    import torch
    import parity as P
    from paper_2606_14782_amd import bacon
    if not wide:
        monkeypatch.setenv("BACON_WIDE", "0")
    L = 20
    wl = _wl(L, 4, 2, 64, 16, 5, "bf16", (700, 2100, 290), (20, 60, 9))
    rng = np.random.default_rng(9)
    sched = [(10 + 4 * l, 30 + 7 * l, 5 + 3 * ((l * 7) % L)) for l in range(L)]
    batches = [bacon.BatchLayout(wl.cu_seqlens, np.asarray(s, np.int32), head_budgets=None if adaptive else
                                 rng.integers(1, 90, (wl.batch, wl.num_kv_heads)).astype(np.int32)) for s in sched]
    xs = [inputs.layer_inputs(wl, l) for l in range(L)]
    qs, ks, vs = ([P.to_dev(x[n], wl) for x in xs] for n in ("q_win", "k", "v"))
    prm = P.params_for(wl, head_alloc=bacon.ALLOC_ADAPTIVE if adaptive else bacon.ALLOC_GIVEN, alloc_floor=0.2)
    a, b = P.make_ctx(wl, prm), P.make_ctx(wl, prm)
    b.bacon_profile_enable(True)
    lses = [a.bacon_window_lse(batches[0], q, k) for q, k in zip(qs, ks)] if lse else None
    a.bacon_begin_prompt(batches[0])
    want = [a.bacon_compress_layer_lse(l, batches[l], qs[l], ks[l], vs[l], lses[l]) if lse else
            a.bacon_compress_layer(l, batches[l], qs[l], ks[l], vs[l]) for l in range(L)]
    b.bacon_begin_prompt(batches[0])
    got = b.bacon_compress_prompt(0, batches[0], qs, ks, vs, lses=lses, layer_batches=batches)
    torch.cuda.synchronize()
    for l in range(L):
        for x, y in zip(got[l], want[l]):
            assert torch.equal(x, y), f"layer {l}"
    assert a.bacon_debug_device_errors() == 0 and b.bacon_debug_device_errors() == 0
    assert ("layer_stages" in b.bacon_profile_read()) == wide


def _budgets_by_counting(B, cu, W, budgets, half, alpha):
    """The adaptive allocation's budgets by sorting the pooled scores, pooled
    in float32 in position order as the GPU does."""
    import numpy as np
    H = B.shape[0]
    out = []
    for b, K in enumerate(budgets):
        x = B[:, cu[b]:cu[b + 1] - W]
        nc = x.shape[1]
        if nc <= K:
            out.append([K] * H)
            continue
        A = np.zeros_like(x)
        cnt = np.zeros(nc, np.float32)
        for o in range(-half, half + 1):
            lo, hi = max(0, -o), min(nc, nc - o)
            A[:, lo:hi] += x[:, lo + o:hi + o]
            cnt[lo:hi] += 1
        A = A / cnt
        f = int(min(float(K), np.floor(float(np.float32(alpha)) * K)))
        rest = []
        for h in range(H):
            order = np.lexsort((np.arange(nc), -A[h]))[f:]
            rest += [(-A[h, i], h, i) for i in order]
        rest.sort()
        kh = [f] * H
        for _, h, _i in rest[:H * (K - f)]:
            kh[h] += 1
        out.append(kh)
    return np.array(out, np.int32)


@pytest.mark.parametrize("hkv,lens,budgets", [
    (1, (64, 2080, 33), (10, 100, 40)),          # one head; a sequence that keeps everything
    (5, (2047, 4130), (17, 400)),
    (32, (1000, 6200), (50, 300)),
])
@pytest.mark.parametrize("values", ["spread", "ties", "negative", "constant"])
@pytest.mark.parametrize("alpha", [0.0, 0.2, 1.0])
def test_allocation(hkv, lens, budgets, values, alpha):
    """bacon_allocate_heads against sorting, exactly: keys spread over many
    bins, thousands of ties in the boundary bin, negative values (which share
    the histogram's lowest bin), and one constant."""
    import numpy as np
    import torch
    import parity as P
    from paper_2606_14782_amd import bacon
    wl = _wl(1, hkv, hkv, 64, 16, 5, "bf16", lens, budgets)
    rng = np.random.default_rng(hkv * 100 + len(values))
    T = wl.total_tokens
    B = rng.random((hkv, T), dtype=np.float32) ** 3
    if values == "ties":
        B = np.round(B * 4).astype(np.float32) / 4
    elif values == "negative":
        B -= 0.9
    elif values == "constant":
        B = np.full_like(B, 0.25)
    ctx = P.make_ctx(wl, P.params_for(wl, alloc_floor=alpha))
    batch = bacon.BatchLayout(wl.cu_seqlens, wl.budgets_arr)
    got = ctx.bacon_allocate_heads(batch, torch.from_numpy(B).cuda()).cpu().numpy()
    again = ctx.bacon_allocate_heads(batch, torch.from_numpy(B).cuda()).cpu().numpy()
    want = _budgets_by_counting(B, wl.cu_seqlens, wl.window, wl.budgets, wl.pool_kernel // 2, alpha)
    assert np.array_equal(got, again)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("lens,budgets,kw", [
    ((33, 2048, 2081), (4, 300, 90), {}),                       # one candidate; a segment and a window past it
    ((4097, 700), (1500, 40), {"pool_mode": 2}),                # pooling before calibration over a segment's edge
    ((6300,), (3100,), {}),                                     # lists beyond one workgroup: every position
])
def test_split_segments(lens, budgets, kw):
    """The split calls over several segments against the oracle (scores, V and
    lambda of every position, the kept sets)."""
    wl = _wl(6, 4, 2, 64, 32, 7, "bf16", lens, budgets)
    TP.run_case("split-segments", wl, gpu_kw=kw, orc_kw=dict(kw), fused=False)


@pytest.mark.parametrize("wide", [True, False])
@pytest.mark.parametrize("window,dtype", [(32, "bf16"), (8, "fp32")])
def test_boundary_far_below_the_maximum(window, dtype, wide, monkeypatch):
    """A sink that takes nearly all attention and thousands of positions within
    a few per cent of each other, 17 octaves below it: the boundary bin of B
    overflows the lists and lies below the octaves that the whole-sequence
    threshold bins first.  Lambda against the set and the moments (float64) of
    the call's own B and V."""
    import numpy as np
    import torch
    import parity as P
    from paper_2606_14782_amd import bacon
    if not wide:
        monkeypatch.setenv("BACON_WIDE", "0")
    wl = _wl(2, 4, 2, 64, window, 5, dtype, (6300, 3100), (1300, 700))
    batch = bacon.BatchLayout(wl.cu_seqlens, wl.budgets_arr)
    d, T, H = wl.head_dim, wl.total_tokens, wl.num_kv_heads
    ctx = P.make_ctx(wl)
    cap = [torch.zeros(s, device="cuda") for s in ((2, H, T), (2, H, T), (2, 2, H))]
    ctx.bacon_debug_capture(*cap)
    ctx.bacon_begin_prompt(batch)
    for layer in range(2):
        rng = np.random.default_rng(layer)
        u = rng.standard_normal(d).astype(np.float32)
        u /= np.linalg.norm(u)
        q = 4 * u + 0.05 * rng.standard_normal((wl.batch * window, wl.num_q_heads, d)).astype(np.float32)
        k = 0.01 * rng.standard_normal((T, H, d)).astype(np.float32)
        for b in range(wl.batch):
            k[wl.cu_seqlens[b]] = 3.2 * np.sqrt(d) * u          # logit 12.8 against 0
        q, k = (P.to_dev(inputs.round_bf16(x), wl) for x in (q, k))
        ctx.bacon_compress_layer(layer, batch, q, k, k)
    torch.cuda.synchronize()
    B, V, lam = (x.cpu().numpy().astype(np.float64) for x in cap)
    for layer in range(2):
        for b, (s0, s1) in enumerate(P.seq_slices(wl)):
            nc = s1 - s0 - window
            for h in range(H):
                bb, vv = B[layer, h, s0:s0 + nc], V[layer, h, s0:s0 + nc]
                m = np.lexsort((np.arange(nc), -bb))[:2 * wl.budgets[b]]
                want = bb[m].std() / (vv[m].std() + 1e-12)
                # moments in double of the same float32 values, lambda rounded to float32
                assert abs(lam[layer, b, h] - want) <= 1e-6 * want, (layer, b, h)


def _calibrate64(B, Q, cu, W, budgets, radius, rho, pool_half, pool_mode):
    """First-layer calibration of any B and Q in float64: S, lambda, E, V.  The
    scale-matching set is taken from the float32 B (score descending, position
    ascending); V enters lambda as the float32 the GPU keeps."""
    import numpy as np
    H, T = B.shape
    E = np.maximum(Q - B, 0).astype(np.float32).astype(np.float64)
    S, V, lam = np.zeros((H, T)), np.zeros((H, T)), np.zeros((len(budgets), H))

    def box(x, r):
        c = np.concatenate([[0.0], np.cumsum(x)])
        i = np.arange(len(x))
        lo, hi = np.maximum(0, i - r), np.minimum(len(x), i + r + 1)
        return (c[hi] - c[lo]) / (hi - lo)
    for b, K in enumerate(budgets):
        sl, nc = slice(cu[b], cu[b + 1]), cu[b + 1] - cu[b] - W
        for h in range(H):
            bb = B[h, sl].astype(np.float64)
            v = E[h, sl] + box(E[h, sl], radius)
            M = min(int(rho * K), nc)
            m = np.lexsort((np.arange(nc), -bb[:nc]))[:M]
            lam[b, h] = bb[m].std() / (v[m].std() + 1e-12)
            if pool_mode == 2:
                bb[:nc] = box(bb[:nc], pool_half)
            V[h, sl], S[h, sl] = v, bb + lam[b, h] * v
    return S, lam, E, V


@pytest.mark.parametrize("lens,budgets,keep", [
    ((1500, 33), (400, 9), 100),           # the boundary among 1368 negative entries, on the lists
    ((2300,), (150,), 200),                # lists over two segments
    ((5000,), (2150,), 4200),              # lists beyond one workgroup: 768 negative entries
    ((6000, 4500), (2500, 1000), 300),     # thousands of them
])
def test_calibrate_on_signed_scores(lens, budgets, keep):
    """bacon_calibrate takes any B: negative values, which share the lowest bin of
    the histogram, are ranked over their whole keys (ties by position)."""
    import numpy as np
    import torch
    import parity as P
    from paper_2606_14782_amd import bacon
    wl = _wl(1, 2, 2, 64, 32, 5, "bf16", lens, budgets)
    rng = np.random.default_rng(len(lens) + keep)
    B = -np.exp(rng.uniform(np.log(1e-3), np.log(30.0), (2, wl.total_tokens))).astype(np.float32)
    B[:, ::7] = np.round(B[:, ::7] * 8) / 8            # ties
    for b, n in enumerate(lens):
        pos = rng.permutation(n - wl.window)[:keep]
        B[:, wl.cu_seqlens[b] + pos] *= -1
    Q = (B + rng.standard_normal(B.shape) * 0.2).astype(np.float32)
    batch = bacon.BatchLayout(wl.cu_seqlens, wl.budgets_arr)
    ctx = P.make_ctx(wl)
    ctx.bacon_begin_prompt(batch)
    got = ctx.bacon_calibrate(0, batch, torch.from_numpy(B).cuda(), torch.from_numpy(Q).cuda(), True, True)
    want = _calibrate64(B, Q, wl.cu_seqlens, wl.window, budgets, 5, 2.0, 2, 0)
    for name, w in zip(("S", "lambda", "E", "V"), want):
        # float32 V (a sum of 11 and two more terms): below 1e-6 of its values
        g = got[name].cpu().numpy()
        assert np.abs(g - w).max() <= 1e-5 * np.abs(w).max(), name


@pytest.mark.parametrize("pool_mode", [0, 2])
@pytest.mark.parametrize("over", [("S", "E", None), ("E", "S", None), ("V", "E", "S"), (None, "V", "S")])
def test_calibrate_in_place(pool_mode, over):
    """bacon_calibrate with outputs over its inputs (over: what B's buffer, Q's
    buffer and a third one receive): the same as into buffers of their own, over
    several segments and with lists beyond one workgroup, whose scale-matching set
    is taken from every position's B."""
    import ctypes
    import torch
    import parity as P
    from paper_2606_14782_amd import bacon
    wl = _wl(2, 4, 2, 64, 32, 7, "bf16", (6300, 2100, 40), (3100, 200, 4))
    batch = bacon.BatchLayout(wl.cu_seqlens, wl.budgets_arr)
    g = torch.Generator(device="cuda").manual_seed(5)
    B = torch.rand(2, wl.total_tokens, device="cuda", generator=g) ** 3
    Q = torch.rand(2, wl.total_tokens, device="cuda", generator=g) ** 3
    a, c = (P.make_ctx(wl, P.params_for(wl, pool_mode=pool_mode)) for _ in range(2))
    a.bacon_begin_prompt(batch)
    c.bacon_begin_prompt(batch)
    ptr = lambda t: None if t is None else ctypes.c_void_p(t.data_ptr())
    for layer in range(2):
        want = a.bacon_calibrate(layer, batch, B, Q, want_E=True, want_V=True)
        bufs = [B.clone(), Q.clone(), torch.empty_like(B)]
        out = {n: bufs[i] for i, n in enumerate(over) if n}
        lam = torch.empty_like(want["lambda"])
        S = out.get("S", torch.empty_like(B))
        bacon._check(bacon.lib().bacon_calibrate(
            c._h, layer, ctypes.byref(batch.c), ptr(bufs[0]), ptr(bufs[1]), ptr(S), ptr(lam),
            ptr(out.get("E")), ptr(out.get("V")), bacon._stream()))
        torch.cuda.synchronize()
        assert torch.equal(lam, want["lambda"])
        for n, t in dict(out, S=S).items():
            assert torch.equal(t, want[n]), (layer, n)


@pytest.mark.parametrize("adaptive", [False, True])
def test_prompts_of_changing_batches(adaptive):
    """begin_prompt clears the rows of its batch in a workspace of any content:
    prompts of one and three sequences in a context for five give what contexts
    of their own give."""
    import torch
    import parity as P
    from paper_2606_14782_amd import bacon
    lens, budgets = (900, 2100, 300), (20, 150, 9)
    prm = dict(head_alloc=bacon.ALLOC_ADAPTIVE) if adaptive else {}
    full = _wl(6, 4, 2, 64, 16, 5, "bf16", lens, budgets)
    big = bacon.Context(6, 4, 2, 64, 16, 5, 2 * full.total_tokens, "bf16", P.params_for(full, **prm))
    for n in (1, 3, 1, 2):
        wl = _wl(6, 4, 2, 64, 16, 5, "bf16", lens[:n], budgets[:n])
        big.workspace.fill_(0x7f)
        batch = bacon.BatchLayout(wl.cu_seqlens, wl.budgets_arr)
        xs = [inputs.layer_inputs(wl, l) for l in range(6)]
        qs, ks, vs = ([P.to_dev(x[k], wl) for x in xs] for k in ("q_win", "k", "v"))
        own = P.make_ctx(wl, P.params_for(wl, **prm))
        for ctx in (own, big):
            ctx.bacon_begin_prompt(batch)
        want = own.bacon_compress_prompt(0, batch, qs, ks, vs)
        got = big.bacon_compress_prompt(0, batch, qs, ks, vs)
        torch.cuda.synchronize()
        for l in range(6):
            for x, y in zip(got[l], want[l]):
                assert torch.equal(x, y), (n, l)
        assert big.bacon_debug_device_errors() == 0


@pytest.mark.parametrize("hq,hkv,d,window,dtype,lens", [
    (7, 1, 128, 32, "bf16", (513, 2049, 97)),        # 224 rows
    (12, 1, 64, 16, "bf16", (4100, 33)),             # 192 rows, a window other than 32 queries
    (4, 1, 128, 32, "fp32", (700, 3000)),            # 128 rows of fp32
    (15, 1, 64, 8, "fp32", (2049, 64)),              # 120, in a padded row tile
])
def test_given_normalisers_on_either_pass(hq, hkv, d, window, dtype, lens):
    """With the normalisers given, layer calls of many window rows take the
    streaming pass 2 and the prompt call the wide one: the same bits."""
    import torch
    import parity as P
    from paper_2606_14782_amd import bacon
    wl = _wl(4, hq, hkv, d, window, 7, dtype, lens, [max(1, n // 10) for n in lens])
    batch = bacon.BatchLayout(wl.cu_seqlens, wl.budgets_arr)
    xs = [inputs.layer_inputs(wl, l) for l in range(4)]
    qs, ks, vs = ([P.to_dev(x[n], wl) for x in xs] for n in ("q_win", "k", "v"))
    a, b = P.make_ctx(wl), P.make_ctx(wl)
    lses = [a.bacon_window_lse(batch, q, k) for q, k in zip(qs, ks)]
    shape = (4, hkv, wl.total_tokens)
    caps = [[torch.zeros(s, device="cuda") for s in (shape, shape, (4, wl.batch, hkv))] for _ in range(2)]
    for ctx, cap in zip((a, b), caps):
        ctx.bacon_profile_enable(True)
        ctx.bacon_debug_capture(*cap)
        ctx.bacon_begin_prompt(batch)
    want = [a.bacon_compress_layer_lse(l, batch, qs[l], ks[l], vs[l], lses[l]) for l in range(4)]
    got = b.bacon_compress_prompt(0, batch, qs, ks, vs, lses=lses)
    torch.cuda.synchronize()
    for l in range(4):
        for x, y in zip(got[l], want[l]):
            assert torch.equal(x, y), f"layer {l}"
    assert torch.equal(caps[0][0], caps[1][0]) and torch.equal(caps[0][2], caps[1][2])   # B, lambda
    assert "window_score_calib" in a.bacon_profile_read() and "layer_stages" in b.bacon_profile_read()
