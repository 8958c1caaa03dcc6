"""Every form that a kernel route accepts against the float64 oracle, at the sizes where the route can go wrong:
edges of tiles and chunks, remainders, the smallest and largest of its range, padded strides."""
import numpy as np
import pytest
import torch

from oracle import uncomp_oracle as O
from paper_2410_03090_amd import synth
from tests._util import to_f64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    from paper_2410_03090_amd import binding
    c = binding.Context(0, 256 << 20)
    yield c
    c.close()


def _padded(t, extra):
    """The same values with rows `extra` elements further apart."""
    big = torch.full((*t.shape[:-1], t.shape[-1] + extra), 7.0, dtype=t.dtype, device=t.device)
    view = big[..., : t.shape[-1]]
    view.copy_(t)
    return view


# 64-wide heads and row groups (more than 256 query rows per KV head) through the matrix-core scoring kernels; windows of
# under eight rows stay on the plain-arithmetic ones.  Scores are held to 2e-5 relative as everywhere: fp32 logits of
# magnitude <= ~16 carry ~1e-6 relative error into exp().
@pytest.mark.parametrize("D,G,N,w", [
    (64, 1, 17, 16), (64, 2, 65, 8), (64, 4, 2049, 32), (64, 4, 4161, 64), (64, 8, 2500, 16), (64, 8, 700, 64),
    (64, 3, 300, 5), (128, 8, 4160, 64), (128, 16, 2111, 32), (128, 5, 1000, 64), (128, 64, 530, 8), (128, 17, 333, 16),
    (128, 1, 1500, 512), (128, 2, 65, 48)])
def test_score_head_widths_and_row_groups(ctx, D, G, N, w):
    cfg = synth.tiny_config(dtype="bf16", B=2, H=2, G=G, N=N, D=D, w=w, rank_lo=2, rank_hi=48)
    K, V, Q = synth.gen_all(cfg, seed0=N + G)
    ref = O.window_score(to_f64(Q[0]), to_f64(K[0]), G=G, pool=7)
    Qd, Kd = Q[0].to(DEV), K[0].to(DEV)
    np.testing.assert_allclose(ctx.window_score(Qd, Kd, G=G, pool=7).cpu().numpy(), ref, rtol=2e-5)
    np.testing.assert_allclose(ctx.window_score(Qd, _padded(Kd, 24), G=G, pool=7).cpu().numpy(), ref, rtol=2e-5)
    lse = torch.from_numpy(O.window_lse(to_f64(Q[0]), to_f64(K[0]), G).astype(np.float32)).to(DEV)
    np.testing.assert_allclose(ctx.window_score(Qd, Kd, G=G, pool=7, lse=lse).cpu().numpy(), ref, rtol=2e-5)


# Gram sums of 64-wide heads on the matrix cores: 64-token steps in two halves, N around the steps and the 128-token
# chunk granularity.  The tolerances are those of the 128-wide kernel's tests (fp32 sums of exact products).
@pytest.mark.parametrize("N", [2, 31, 33, 64, 65, 127, 129, 1000, 4099, 9001])
def test_entropy_64_wide_heads(ctx, N):
    g = torch.Generator().manual_seed(N)
    X = (torch.randn(5, N, 12, generator=g) @ torch.randn(5, 12, 64, generator=g) / 12 +
         0.1 * torch.randn(5, N, 64, generator=g) + 0.05).to(torch.bfloat16)
    for flags in (O.DEFAULT_FLAGS, 0):
        Href, eref = O.head_entropy(to_f64(X), k_trunc=32, flags=flags)
        for Xd in (X.to(DEV), _padded(X.to(DEV), 8)):
            H, eig = ctx.head_entropy(Xd, k_trunc=32, flags=flags, want_eig=True)
            np.testing.assert_allclose(H.cpu().numpy(), Href, rtol=1e-4, atol=5e-5)
            np.testing.assert_allclose(eig.cpu().numpy(), eref, rtol=0, atol=2e-5)


# The 64-wide eigen stage knows 64 eigenvalues: more are asked for than there are, and lanes per eigenvalue change at 32.
# 2e-7: entropies and shares rounded to fp32 (2^-24 of values up to 4.2) on top of brackets of 2.9e-10.
@pytest.mark.parametrize("k", [1, 32, 33, 64, 65, 128])
def test_entropy_64_wide_truncation(ctx, k):
    g = torch.Generator().manual_seed(k)
    X = torch.randint(-3, 4, (9, 200, 64), generator=g).to(torch.bfloat16)      # exact Grams
    X[0, :, 32:] = X[0, :, :32]                                                 # rank 32
    for flags in (O.DEFAULT_FLAGS, 0):
        Href, eref = O.head_entropy(to_f64(X), k_trunc=k, flags=flags)
        H, eig = ctx.head_entropy(X.to(DEV), k_trunc=k, flags=flags, want_eig=True)
        assert torch.equal(H, ctx.head_entropy(X.to(DEV), k_trunc=k, flags=flags))
        np.testing.assert_allclose(H.cpu().numpy(), Href, rtol=0, atol=5e-7)
        np.testing.assert_allclose(eig.cpu().numpy(), eref[:, :64], rtol=0, atol=2e-8)


# Matrices of low rank: long runs of zero eigenvalues, along which the terms of the Sturm recurrence shrink by 2^-32 a step.
# The inputs are small whole numbers, so the Gram is exact.  The last bracket of an eigenvalue is 2.9e-10 wide: its middle is
# off by half of that, and a zero eigenvalue is exactly zero.  The rest of the entropy's error is rounding to fp32 (2.4e-7).
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("rank", [1, 4, 8, 40])
def test_entropy_low_rank(ctx, D, rank):
    g = torch.Generator().manual_seed(rank)
    U = torch.randint(-1, 2, (2, 64, rank), generator=g).double()
    X = U @ torch.randint(-1, 2, (2, rank, D), generator=g).double()
    X[1] = 3.0 * torch.eye(D, dtype=torch.float64)[torch.arange(64) % rank]      # `rank` equal eigenvalues, not centred
    for dtype in (torch.bfloat16, torch.float32):
        for flags in (O.DEFAULT_FLAGS, O.DEFAULT_FLAGS & ~O.FLAG_CENTER):
            Href, eref = O.head_entropy(X.numpy(), k_trunc=32, flags=flags)
            Xd = X.to(dtype).to(DEV)
            H, eig = ctx.head_entropy(Xd, k_trunc=32, flags=flags, want_eig=True)
            np.testing.assert_allclose(eig.cpu().numpy(), eref, rtol=1.2e-7, atol=2e-10)
            assert bool((eig.cpu().numpy()[eref < 1e-12] == 0.0).all())
            for h in (H, ctx.head_entropy(Xd, k_trunc=32, flags=flags)):         # all eigenvalues and the 32 largest alone
                np.testing.assert_allclose(h.cpu().numpy(), Href, rtol=0, atol=2.5e-7)


# Chunks of the scoring passes: from one 256-token round to many, a last chunk that holds fewer tokens than the window
# or than a tile, logits that grow along the prompt (the running reference of a row must follow them).
@pytest.mark.parametrize("H,G,N,w", [(1, 4, 256, 32), (1, 4, 257, 32), (2, 2, 1025, 64), (8, 4, 8200, 32), (3, 8, 40009, 32),
                                     (1, 1, 2049, 16)])
def test_score_chunks(ctx, H, G, N, w):
    cfg = synth.tiny_config(dtype="bf16", B=1, H=H, G=G, N=N, w=w, rank_lo=2, rank_hi=24)
    K, V, Q = synth.gen_all(cfg, seed0=N)
    ramp = torch.linspace(0.02, 3.0, N).view(1, 1, N, 1)
    for k in (K[0], (K[0].float() * ramp).to(torch.bfloat16)):
        ref = O.window_score(to_f64(Q[0]), to_f64(k), G=G, pool=7)
        got = ctx.window_score(Q[0].to(DEV), k.to(DEV), G=G, pool=7).cpu().numpy()
        # logits up to three times those of the other tests: exp() carries three times their relative error
        np.testing.assert_allclose(got, ref, rtol=6e-5, atol=1e-12)


# fp32 logits on the matrix cores: fp32 inputs, and bf16 windows without a cut into 16-row blocks.  128-token tiles and
# 16-row blocks with remainders, windows of eight in pairs and alone, rows split over workgroups and not, the widest R.
@pytest.mark.parametrize("dtype,D,H,G,N,w", [
    ("f32", 128, 2, 1, 9, 8), ("f32", 128, 1, 4, 160, 32), ("f32", 128, 2, 2, 161, 8), ("f32", 64, 2, 3, 1025, 8),
    ("f32", 128, 2, 3, 700, 20), ("f32", 64, 1, 8, 2333, 64), ("f32", 128, 8, 4, 1024, 32), ("f32", 128, 1, 7, 290, 33),
    ("f32", 128, 1, 1, 1500, 512), ("f32", 128, 64, 8, 1100, 16), ("bf16", 128, 2, 3, 700, 20), ("bf16", 64, 2, 5, 333, 9)])
def test_score_fp32_logits(ctx, dtype, D, H, G, N, w):
    cfg = synth.tiny_config(dtype=dtype, B=1, H=H, G=G, N=N, D=D, w=w, rank_lo=2, rank_hi=48)
    K, V, Q = synth.gen_all(cfg, seed0=N + G)
    ref = O.window_score(to_f64(Q[0]), to_f64(K[0]), G=G, pool=5)
    Qd, Kd = Q[0].to(DEV), K[0].to(DEV)
    # as above: fp32 logits of magnitude <= ~16
    np.testing.assert_allclose(ctx.window_score(Qd, Kd, G=G, pool=5).cpu().numpy(), ref, rtol=2e-5)
    np.testing.assert_allclose(ctx.window_score(Qd, _padded(Kd, 24), G=G, pool=5).cpu().numpy(), ref, rtol=2e-5)
    lse = torch.from_numpy(O.window_lse(to_f64(Q[0]), to_f64(K[0]), G).astype(np.float32)).to(DEV)
    np.testing.assert_allclose(ctx.window_score(Qd, Kd, G=G, pool=5, lse=lse).cpu().numpy(), ref, rtol=2e-5)


# Logits beyond the numbers, on every scoring route: -inf is a token without weight (whole tiles of them, the first ones
# among them), +inf and NaN leave a row without a normaliser, and its KV head without scores, whichever chunk they fall in.
@pytest.mark.parametrize("dtype,D,G,w,plain", [
    ("bf16", 128, 4, 16, False), ("bf16", 64, 4, 16, False), ("bf16", 128, 16, 32, False), ("bf16", 128, 3, 20, False),
    ("bf16", 128, 4, 1, False), ("f32", 128, 4, 16, False), ("f32", 64, 2, 8, False), ("f32", 128, 4, 4, False),
    ("f32", 128, 2, 1, False), ("bf16", 128, 4, 16, True), ("f32", 64, 4, 16, True)])
@pytest.mark.parametrize("N", [331, 5000])
def test_score_infinities_and_nan(ctx, dtype, D, G, w, plain, N):
    cfg = synth.tiny_config(dtype=dtype, B=1, H=5, G=G, N=N, D=D, w=w, rank_lo=2, rank_hi=48)
    K, V, Q = synth.gen_all(cfg, seed0=N)
    K, Q = K[0].clone(), Q[0].clone()
    Q[..., 5] = 0.5                                                 # every row's logit takes the sign of the key's entry
    K[0, 0, 2 * N // 3, 5] = float("inf")
    K[0, 1, :70, 5] = K[0, 1, 150:290, 5] = float("-inf")
    K[0, 2, 7, 5] = float("nan")
    K[0, 3, N // 2, 5] = K[0, 3, N // 2 + 1, 5] = float("inf")
    with np.errstate(invalid="ignore"):
        ref = O.window_score(to_f64(Q), to_f64(K), G=G, pool=7)
    assert [bool(np.isnan(ref[0, h]).all()) for h in range(5)] == [True, False, True, True, False]
    ctx.set_kernel_path(plain)
    try:
        got = ctx.window_score(Q.to(DEV), K.to(DEV), G=G, pool=7).cpu().numpy()
    finally:
        ctx.set_kernel_path(False)
    assert not np.isfinite(got[0, [0, 2, 3]]).any()                 # (NaN; -inf where the pool reaches past the prefix)
    np.testing.assert_allclose(got[0, [1, 4]], ref[0, [1, 4]], rtol=2e-5)        # as everywhere


# Gram of fp32 matrices with its tiles over nine, three and one workgroup per chunk (few, more and many matrices).
@pytest.mark.parametrize("n_mat,N", [(1, 2), (3, 65), (8, 1024), (57, 130), (171, 70)])
def test_entropy_fp32_tile_split(ctx, n_mat, N):
    g = torch.Generator().manual_seed(N)
    X = torch.randn(n_mat, N, 12, generator=g) @ torch.randn(n_mat, 12, 128, generator=g) / 12 + \
        0.1 * torch.randn(n_mat, N, 128, generator=g) + 0.05
    Href, eref = O.head_entropy(to_f64(X), k_trunc=32, flags=O.DEFAULT_FLAGS)
    H, eig = ctx.head_entropy(X.to(DEV), k_trunc=32, flags=O.DEFAULT_FLAGS, want_eig=True)
    np.testing.assert_allclose(H.cpu().numpy(), Href, rtol=1e-4, atol=5e-5)
    np.testing.assert_allclose(eig.cpu().numpy(), eref, rtol=0, atol=2e-5)


def _decode_names(c):
    """Kernels of the last decode step of a context that profiles, in order (the read clears them)."""
    return [name for name, _ in c.profile_read()]


HEAD, SPREAD, TWO = ["decode_head"], ["decode_split"], ["decode_attend_wave", "decode_update"]


# The decode step of many heads in one kernel: eight, four and two waves per head, lengths around the 16-row tiles and the
# waves' turns, evictions, growth and full caches, and a key far down the cache whose logit is 34 above all others (the
# waves' reference has to follow it).  Tolerances of the step as everywhere (_check_step).
@pytest.mark.parametrize("n_heads,G,cap,w", [(256, 4, 300, 8), (257, 7, 270, 3), (1024, 8, 290, 16), (1030, 1, 150, 5),
                                             (256, 2, 16, 4), (2050, 8, 270, 8), (2048, 3, 100, 4), (300, 4, 1700, 8),
                                             (256, 8, 1990, 8)])
def test_decode_many_heads(ctx, n_heads, G, cap, w):
    from tests.test_gpu_decode import D, _check_step, _random_state
    edges = [0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, cap - 1, cap, min(cap, 260), min(cap, 200)]
    lens = [min(cap, edges[h % len(edges)]) for h in range(n_heads)]
    pos0 = [cap + 50 + h % 90 for h in range(n_heads)]
    st = _random_state(n_heads, cap, lens, pos0, torch.bfloat16, seed=cap, w=w)
    budget = torch.tensor([(h * 37) % (cap + 20) if h % 3 else lens[h] for h in range(n_heads)], dtype=torch.int32)
    g = torch.Generator().manual_seed(G)
    heads = sorted(set(range(0, n_heads, n_heads // 48)) | set(range(n_heads - len(edges), n_heads)))
    swaps = 0
    for t in range(2):
        q = torch.randn(n_heads, G, D, generator=g).to(torch.bfloat16)
        kn, vn = (torch.randn(n_heads, D, generator=g).to(torch.bfloat16) for _ in range(2))
        for h in range(0, n_heads, 2):
            if lens[h] > 150:
                q0 = q[h, 0].float()
                st.Kc[h, lens[h] - 2 - t] = (q0 * (34.0 * D ** 0.5 / float(q0 @ q0))).to(torch.bfloat16).to(DEV)
        pos = torch.tensor([p + t for p in pos0], dtype=torch.int32)
        before = st.host()
        out, ev = ctx.decode_step(q.to(DEV), kn.to(DEV), vn.to(DEV), pos.to(DEV), budget.to(DEV), w, st.Kc, st.Vc, st.idx,
                                  st.cum, st.ln)
        torch.cuda.synchronize()
        swaps += _check_step(before, st.host(), out.cpu().numpy(), ev.cpu().numpy(), q, kn, vn, pos.numpy(),
                             budget.numpy(), w, cap, heads=heads)
    assert swaps <= 2                               # near ties at fp32 resolution, each checked to be one


# Logits at the end of the range and beyond it: the one-kernel step of many heads gives what the step of fewer heads gives for
# the same heads (one kernel too for short caches; spread over workgroups; two kernels), and what the oracle gives where that is
# finite.  The infinity and the NaN lie in the first part of a head's rows and in a later one.
@pytest.mark.parametrize("cap,few,form,at", [(60, 8, HEAD, 37), (400, 8, SPREAD, 37), (400, 8, SPREAD, 301), (800, 136, TWO, 37),
                                             (800, 136, TWO, 700)])
def test_decode_many_heads_extreme_logits(ctx, cap, few, form, at):
    from tests.test_gpu_decode import D, State, _check_step, _random_state
    n_heads, G, w = 256, 4, 4
    lens, pos0 = [cap - 1 - h % 7 for h in range(n_heads)], [cap + 140] * n_heads
    st = _random_state(n_heads, cap, lens, pos0, torch.bfloat16, seed=3, w=w)
    g = torch.Generator().manual_seed(4)
    q = torch.rand(n_heads, G, D, generator=g) + 0.5
    kn, vn = torch.randn(n_heads, D, generator=g), torch.randn(n_heads, D, generator=g).to(torch.bfloat16)
    kinds = ["all below -1e30", "one +inf", "some -inf", "one NaN"]
    row = torch.arange(1, cap + 1).view(1, cap, 1)
    q[0::4], kn[0::4] = 1e16 * q[0::4], -4e16                       # logits of -1e33 and less, one or more per cent apart
    st.Kc[0::4] = (-1e16 * (1 + 0.02 * row)).to(torch.bfloat16).expand(n_heads // 4, cap, D).to(DEV)
    st.Kc[1::4, at, 5] = float("inf")
    st.Kc[2::4, ::3, 9] = float("-inf")
    st.Kc[3::4, at - 26, 0] = float("nan")
    q, kn = q.to(torch.bfloat16), kn.to(torch.bfloat16)
    pos, budget = torch.tensor(pos0, dtype=torch.int32), torch.full((n_heads,), cap, dtype=torch.int32)
    before = st.host()
    part = State(*(t[:few].clone() for t in (st.Kc, st.Vc, st.idx, st.cum, st.ln)))
    args = [t.to(DEV) for t in (q, kn, vn, pos, budget)]
    ctx.profile(True)
    try:
        out, ev = ctx.decode_step(*args, w, st.Kc, st.Vc, st.idx, st.cum, st.ln)
        out8, ev8 = ctx.decode_step(*(t[:few].contiguous() for t in args), w, part.Kc, part.Vc, part.idx, part.cum, part.ln)
        torch.cuda.synchronize()
        assert _decode_names(ctx) == HEAD + form
    finally:
        ctx.profile(False)
    # both sum in fp32 over the same rows, in another order: the tolerances of _check_step
    np.testing.assert_allclose(out[:few].cpu().numpy(), out8.cpu().numpy(), rtol=0, atol=1e-4)
    np.testing.assert_allclose(st.cum[:few].cpu().numpy(), part.cum.cpu().numpy(), rtol=2e-5, atol=2e-6)
    finite = [h for h in range(n_heads) if h % 4 in (0, 2)]
    seen = [h for h in finite if h < few]
    assert torch.equal(ev[seen], ev8[seen]) and torch.equal(st.ln[:few], part.ln)
    for h in range(n_heads):
        assert bool(torch.isfinite(out[h]).all()) == (h % 4 in (0, 2)), kinds[h % 4]
        assert bool(torch.isnan(out[h]).all()) == (h % 4 in (1, 3)), kinds[h % 4]
    assert _check_step(before, st.host(), out.cpu().numpy(), ev.cpu().numpy(), q, kn, vn, pos.numpy(), budget.numpy(), w, cap,
                       heads=finite[:64]) == 0


# The attention output needs a float's alignment and no more, on each route of the step.
@pytest.mark.parametrize("n_heads,G,cap,form", [(3, 4, 150, HEAD), (3, 16, 150, TWO), (256, 8, 150, HEAD), (3, 4, 400, SPREAD),
                                                (3, 8, 400, SPREAD), (130, 4, 800, TWO), (130, 8, 800, TWO)])
def test_decode_output_at_any_float(ctx, n_heads, G, cap, form):
    from tests.test_gpu_decode import D, State, _random_state
    w = 4
    st = _random_state(n_heads, cap, [cap - h % 50 for h in range(n_heads)], [cap + 150] * n_heads, torch.bfloat16, seed=G, w=w)
    g = torch.Generator().manual_seed(G)
    q = torch.randn(n_heads, G, D, generator=g).to(torch.bfloat16).to(DEV)
    kn, vn = (torch.randn(n_heads, D, generator=g).to(torch.bfloat16).to(DEV) for _ in range(2))
    pos, budget = (torch.full((n_heads,), v, dtype=torch.int32, device=DEV) for v in (cap + 150, cap))
    outs = []
    ctx.profile(True)
    for off in range(4):
        s = State(*(t.clone() for t in (st.Kc, st.Vc, st.idx, st.cum, st.ln)))
        buf = torch.full((n_heads * G * D + 8,), 7.0, device=DEV)
        out = buf[off:off + n_heads * G * D].view(n_heads, G, D)
        ctx.decode_step(q, kn, vn, pos, budget, w, s.Kc, s.Vc, s.idx, s.cum, s.ln, out=out)
        torch.cuda.synchronize()
        assert bool((buf[:off] == 7.0).all()) and bool((buf[off + n_heads * G * D:] == 7.0).all())
        outs.append(out.clone())
    names = _decode_names(ctx)
    ctx.profile(False)
    assert names == 4 * form
    assert all(torch.equal(outs[0], o) for o in outs[1:])


def _decode_bytes(n_heads, G, cap, wave_rows):
    """Workspace of the two-kernel step with waves of so many rows (regions are rounded up to 256 bytes)."""
    GT = 4 if G <= 4 else (8 if G <= 8 else 16)
    parts = (cap + wave_rows) // wave_rows
    regions = (G * 128, parts * wave_rows * GT, parts * GT * 2, parts * GT * 128)
    return sum((n_heads * r * 4 + 255) // 256 * 256 for r in regions)


# Few heads: 64-row waves, and the 128-row ones of a workspace that only holds their partials; calls that take another form are
# the same in either.
@pytest.mark.parametrize("n_heads,G,cap,form", [(1, 4, 64, HEAD), (3, 8, 64, HEAD), (5, 16, 130, TWO), (8, 4, 1290, SPREAD),
                                                (136, 4, 800, TWO), (130, 8, 769, TWO), (84, 4, 2000, TWO)])
def test_decode_few_heads_both_plans(ctx, n_heads, G, cap, form):
    from paper_2410_03090_amd import binding
    from tests.test_gpu_decode import D, _check_step, _random_state
    fine, coarse = _decode_bytes(n_heads, G, cap, 64), _decode_bytes(n_heads, G, cap, 128)
    assert fine > coarse and binding.Context.decode_workspace_bytes(n_heads, G, cap) == fine
    small = binding.Context(0, coarse)              # too small for 64-row waves
    try:
        for c in (ctx, small):
            lens = [cap - 3 * (h % 40) if h < 40 else cap - h for h in range(n_heads)]
            pos0 = [cap + 50 + h for h in range(n_heads)]
            st = _random_state(n_heads, cap, lens, pos0, torch.bfloat16, seed=cap, w=4)
            budget = torch.tensor([cap - h % 50 for h in range(n_heads)], dtype=torch.int32)
            g = torch.Generator().manual_seed(G)
            q = torch.randn(n_heads, G, D, generator=g).to(torch.bfloat16)
            kn, vn = (torch.randn(n_heads, D, generator=g).to(torch.bfloat16) for _ in range(2))
            pos = torch.tensor(pos0, dtype=torch.int32)
            before = st.host()
            c.profile(True)
            out, ev = c.decode_step(q.to(DEV), kn.to(DEV), vn.to(DEV), pos.to(DEV), budget.to(DEV), 4, st.Kc, st.Vc, st.idx,
                                    st.cum, st.ln)
            torch.cuda.synchronize()
            names = _decode_names(c)
            c.profile(False)
            assert names == form
            assert _check_step(before, st.host(), out.cpu().numpy(), ev.cpu().numpy(), q, kn, vn, pos.numpy(),
                               budget.numpy(), 4, cap) == 0
    finally:
        small.close()


# The two-kernel step in every form: waves of 64, 128 and 256 rows, the update kernel of few (early and not), some and many
# heads, lengths around the waves' parts, evictions and growth.  Sampled heads against the oracle.  (Sizes of other forms, for
# which the workspace is asked all the same, stand beside them.)
@pytest.mark.parametrize("n_heads,G,cap,rows,form", [
    (255, 4, 2300, 256, HEAD), (255, 8, 2300, 256, TWO), (512, 8, 2050, 256, TWO), (1280, 8, 2050, 256, TWO), (300, 4, 4100, 256, TWO),
    (512, 4, 5100, 256, TWO), (1290, 3, 5100, 256, TWO), (8, 8, 3100, 64, SPREAD), (9, 8, 700, 64, SPREAD), (2, 16, 3100, 64, TWO),
    (600, 16, 70, 64, TWO), (255, 7, 900, 128, HEAD), (1300, 16, 200, 128, TWO), (84, 4, 2000, 64, TWO), (100, 4, 2000, 128, TWO),
    (100, 8, 2000, 128, TWO), (150, 8, 1200, 128, TWO), (145, 7, 800, 64, TWO)])
def test_decode_two_kernels(n_heads, G, cap, rows, form):
    from paper_2410_03090_amd import binding
    from tests.test_gpu_decode import D, State, _check_step
    need = binding.Context.decode_workspace_bytes(n_heads, G, cap)
    assert need == _decode_bytes(n_heads, G, cap, rows)
    w, g = 8, torch.Generator(device=DEV).manual_seed(cap + G)
    rand = lambda *sh: torch.randn(*sh, generator=g, device=DEV).to(torch.bfloat16)  # noqa: E731
    edges = [0, 1, rows - 1, rows, rows + 1, 2 * rows - 1, 2 * rows, cap // 2, cap - 1, cap]
    ln = torch.tensor([min(cap, edges[h % len(edges)]) for h in range(n_heads)], dtype=torch.int32, device=DEV)
    budget = torch.where(torch.arange(n_heads, device=DEV) % 3 == 0, ln + 5, ln).to(torch.int32)
    idx = torch.argsort(torch.rand(n_heads, cap + 60, generator=g, device=DEV), dim=1)[:, :cap].to(torch.int32).contiguous()
    cum = torch.rand(n_heads, cap, generator=g, device=DEV) * 2
    st = State(rand(n_heads, cap, D), rand(n_heads, cap, D), idx, cum, ln)
    q, kn, vn = 2 * rand(n_heads, G, D), rand(n_heads, D), rand(n_heads, D)
    pos = torch.full((n_heads,), cap + 100, dtype=torch.int32, device=DEV)
    pick = torch.tensor(sorted(set(range(min(n_heads, 11))) | set(range(n_heads - min(n_heads, 10), n_heads))), device=DEV)
    sample = lambda: State(*(t[pick] for t in (st.Kc, st.Vc, st.idx, st.cum, st.ln))).host()  # noqa: E731
    c = binding.Context(0, need)
    try:
        before, ln0 = sample(), ln.clone()
        c.profile(True)
        out, ev = c.decode_step(q, kn, vn, pos, budget, w, st.Kc, st.Vc, st.idx, st.cum, st.ln)
        torch.cuda.synchronize()
        after = sample()
        assert _decode_names(c) == form
        assert torch.isfinite(out).all() and torch.isfinite(st.cum).all()
        host = [t[pick].cpu() for t in (out, ev, q, kn, vn, pos, budget)]
        assert _check_step(before, after, host[0].numpy(), host[1].numpy(), *host[2:5], host[5].numpy(), host[6].numpy(), w,
                           cap) <= 1
        assert torch.equal(st.ln, torch.where(ev == -1, ln0 + 1, ln0)) and bool((ev >= -1).all())
    finally:
        c.close()


# The step of few heads whose rows are spread over workgroups that the last one merges: 16- and 32-row waves, caches just above
# those that one workgroup takes, the rows where the wave length changes, many parts, the most rows; lengths around the parts,
# heads that grow into a new part, several steps (the counters are left as they were found).
@pytest.mark.parametrize("n_heads,G,cap", [(1, 4, 385), (12, 8, 400), (159, 3, 386), (16, 4, 2048), (12, 4, 2049), (17, 8, 2048),
                                           (8, 4, 3238), (9, 7, 5000), (1, 1, 163840), (2, 8, 81920)])
def test_decode_spread_heads(n_heads, G, cap):
    from paper_2410_03090_amd import binding
    from tests.test_gpu_decode import D, State, _check_step
    w, g = 8, torch.Generator(device=DEV).manual_seed(cap + G)
    rand = lambda *sh: torch.randn(*sh, generator=g, device=DEV).to(torch.bfloat16)  # noqa: E731
    edges = [cap, 0, 1, 126, 127, 128, 129, 254, 255, 256, 257, 383, cap // 2, cap - 1, cap - 2]
    ln = torch.tensor([min(cap, edges[h % len(edges)]) for h in range(n_heads)], dtype=torch.int32, device=DEV)
    budget = torch.where(torch.arange(n_heads, device=DEV) % 3 == 1, ln + 5, ln).to(torch.int32)
    idx = torch.argsort(torch.rand(n_heads, cap + 60, generator=g, device=DEV), dim=1)[:, :cap].to(torch.int32).contiguous()
    cum = torch.rand(n_heads, cap, generator=g, device=DEV) * 2
    st = State(rand(n_heads, cap, D), rand(n_heads, cap, D), idx, cum, ln)
    for h in range(n_heads):                                        # rows that were never written hold anything
        st.Kc[h, int(ln[h]):] = float("nan")
        st.Vc[h, int(ln[h]):] = float("nan")
    pick = torch.tensor(sorted(set(range(min(n_heads, 15))) | {n_heads - 1}), device=DEV)
    sample = lambda: State(*(t[pick] for t in (st.Kc, st.Vc, st.idx, st.cum, st.ln))).host()  # noqa: E731
    c = binding.Context(0, binding.Context.decode_workspace_bytes(n_heads, G, cap))
    c.profile(True)
    try:
        for t in range(3):
            q, kn, vn = 2 * rand(n_heads, G, D), rand(n_heads, D), rand(n_heads, D)
            pos = torch.full((n_heads,), cap + 100 + t, dtype=torch.int32, device=DEV)
            before, ln0 = sample(), st.ln.clone()
            out, ev = c.decode_step(q, kn, vn, pos, budget, w, st.Kc, st.Vc, st.idx, st.cum, st.ln)
            torch.cuda.synchronize()
            assert _decode_names(c) == SPREAD
            host = [x[pick].cpu() for x in (out, ev, q, kn, vn, pos, budget)]
            assert torch.isfinite(out).all()
            assert _check_step(before, sample(), host[0].numpy(), host[1].numpy(), *host[2:5], host[5].numpy(), host[6].numpy(), w,
                               cap) <= 1
            assert torch.equal(st.ln, torch.where(ev == -1, ln0 + 1, ln0))
    finally:
        c.close()


# Which form a call takes, on both sides of every line: 160 heads, 384 rows, 163840 rows in all, what fits in LDS, more than 128
# heads of four parts, eight query heads.
@pytest.mark.parametrize("n_heads,G,cap,form", [
    (1, 4, 384, HEAD), (1, 4, 385, SPREAD), (159, 4, 385, SPREAD), (160, 4, 385, HEAD), (159, 8, 384, HEAD), (40, 4, 4096, SPREAD),
    (40, 4, 4097, TWO), (128, 4, 800, SPREAD), (129, 4, 767, SPREAD), (129, 4, 768, TWO), (159, 1, 959, TWO), (159, 1, 960, SPREAD),
    (150, 8, 895, TWO), (150, 8, 896, SPREAD), (170, 4, 4100, TWO), (1, 9, 64, TWO), (300, 16, 64, TWO)])
def test_decode_forms(n_heads, G, cap, form):
    from paper_2410_03090_amd import binding
    from tests.test_gpu_decode import D, State, _check_step
    g = torch.Generator(device=DEV).manual_seed(cap)
    rand = lambda *sh: torch.randn(*sh, generator=g, device=DEV).to(torch.bfloat16)  # noqa: E731
    full = lambda v: torch.full((n_heads,), v, dtype=torch.int32, device=DEV)  # noqa: E731
    idx = torch.arange(cap, dtype=torch.int32, device=DEV).repeat(n_heads, 1)
    st = State(rand(n_heads, cap, D), rand(n_heads, cap, D), idx, torch.rand(n_heads, cap, generator=g, device=DEV), full(cap))
    q, kn, vn, pos = rand(n_heads, G, D), rand(n_heads, D), rand(n_heads, D), cap + 40
    c = binding.Context(0, binding.Context.decode_workspace_bytes(n_heads, G, cap))
    try:
        one = lambda: State(*(t[-1:] for t in (st.Kc, st.Vc, st.idx, st.cum, st.ln))).host()  # noqa: E731
        before = one()
        c.profile(True)
        out, ev = c.decode_step(q, kn, vn, full(pos), full(cap), 8, st.Kc, st.Vc, st.idx, st.cum, st.ln)
        torch.cuda.synchronize()
        assert _decode_names(c) == form
        host = [t[-1:].cpu() for t in (out, ev, q, kn, vn)]
        assert _check_step(before, one(), host[0].numpy(), host[1].numpy(), *host[2:], np.array([pos]), np.array([cap]), 8, cap) <= 1
    finally:
        c.close()


# The longest cache that 16 query heads may have: the update kernel's three tables fill 64 KiB but for 64 bytes.
def test_decode_longest_cache():
    from paper_2410_03090_amd import binding
    from tests.test_gpu_decode import D, State, _check_step
    G, cap, w = 16, 341 * 128 + 127 - 128, 8
    g = torch.Generator(device=DEV).manual_seed(1)
    rand = lambda *sh: torch.randn(*sh, generator=g, device=DEV).to(torch.bfloat16)  # noqa: E731
    idx = torch.randperm(cap + 50, generator=g, device=DEV)[:cap].to(torch.int32).view(1, cap).contiguous()
    one = lambda v: torch.tensor([v], dtype=torch.int32, device=DEV)  # noqa: E731
    st = State(rand(1, cap, D), rand(1, cap, D), idx, torch.rand(1, cap, generator=g, device=DEV), one(cap))
    q, kn, vn, pos = rand(1, G, D), rand(1, D), rand(1, D), one(cap + 60)
    c = binding.Context(0, binding.Context.decode_workspace_bytes(1, G, cap))
    try:
        before = st.host()
        out, ev = c.decode_step(q, kn, vn, pos, one(cap), w, st.Kc, st.Vc, st.idx, st.cum, st.ln)
        torch.cuda.synchronize()
        assert _check_step(before, st.host(), out.cpu().numpy(), ev.cpu().numpy(), q.cpu(), kn.cpu(), vn.cpu(),
                           pos.cpu().numpy(), np.array([cap]), w, cap) <= 1
    finally:
        c.close()


# Wide-matrix entropy where the Cholesky step retires columns (rank below 128 from few tokens), at one and several splits
# of the sum over the features, ragged token counts, no mean correction.
@pytest.mark.parametrize("N,D,r", [(40, 256, 100), (129, 384, 60), (1000, 2048, 30), (3001, 640, 90)])
def test_matrix_entropy_ranks_and_splits(ctx, N, D, r):
    g = torch.Generator().manual_seed(N)
    X = (torch.randn(N, r, generator=g) @ (torch.randn(r, D, generator=g) * torch.linspace(1.0, 0.05, r)[:, None]) / r + 0.1
         ).to(torch.bfloat16)
    for flags in (O.DEFAULT_FLAGS, O.DEFAULT_FLAGS & ~O.FLAG_CENTER):
        Href, eref = O.head_entropy(to_f64(X[None]), k_trunc=32, flags=flags)
        H, eig = ctx.matrix_entropy(X[None].to(DEV), k_trunc=32, n_iter=12, flags=flags, want_eig=True)
        # as the other tests of this call: the Ritz values of the leading 32 against the fp64 eigenvalues
        np.testing.assert_allclose(H.cpu().numpy(), Href, rtol=1e-4)
        np.testing.assert_allclose(eig.cpu().numpy()[:, :32], eref[:, :32], rtol=0, atol=2e-5)


# Rows split over workgroups: one chunk and many, odd counts, rows that are no multiple of 4 or of a chunk's 2048; budgets from
# none to all; scores with one outlier, with a few hundred ties at the threshold, all equal.  Indices are exact.
@pytest.mark.parametrize("rows,P,w", [(1, 24576, 4), (16, 24577, 3), (17, 32767, 8), (3, 32769, 8), (2, 67591, 32), (1, 131064, 8), (32, 33333, 1), (1, 1_000_003, 64)])
def test_select_rows_over_workgroups(ctx, rows, P, w):
    rng = np.random.default_rng(P)
    N = P + w
    for kind in ("spread", "outlier", "ties", "equal"):
        score = np.exp(rng.standard_normal((1, rows, P)) * 3).astype(np.float32)
        if kind == "outlier":
            score = (1.0 + rng.random((1, rows, P)) * 1e-4).astype(np.float32)
            score[:, :, P // 3] = 1e30
            score[:, :, P // 2] = -1e30
        elif kind == "ties":
            score = (rng.integers(0, P // 300, (1, rows, P)) / 7).astype(np.float32)
        elif kind == "equal":
            score[:] = 0.25
        budget = rng.integers(w, min(P, 60000) + w, (1, rows)).astype(np.int32)
        budget[0, 0] = {"spread": w + 1, "outlier": w + 2, "ties": N, "equal": N - 1}[kind]
        cap = int(budget.max())
        _, _, idx, ln = ctx.select_gather(torch.from_numpy(score).to(DEV), torch.from_numpy(budget).to(DEV), None, None, w, cap, N=N)
        for r in {0, rows // 2, rows - 1}:
            ref = O.select_indices(score[0, r].astype(np.float64), budget[0, r], N, w)
            assert int(ln[0, r]) == len(ref)
            assert np.array_equal(idx[0, r, : len(ref)].cpu().numpy(), ref), (kind, r)


# Rows whose scores crowd (all equal, a few values, all but an outlier within an octave, most of them zero) take about what
# spread ones take: at most twice, half as much again was measured (a million equal scores).
@pytest.mark.parametrize("rows,P", [(8, 24576), (8, 40009), (1, 131072), (2, 1_000_003)])
def test_select_time_of_crowded_rows(ctx, rows, P):
    w, k = 32, P // 2
    g = torch.Generator(device=DEV).manual_seed(P)
    u = torch.rand(1, rows, P, generator=g, device=DEV)
    outlier = 1.0 + 0.9 * u
    outlier[:, :, 5] = 0.0
    kinds = dict(spread=torch.exp(6.0 * u - 3.0), equal=torch.full_like(u, 0.25), outlier=outlier, narrow=outlier ** 0.03,
                 few=torch.floor(300.0 * u) / 7.0, zeros=torch.where(u < 0.9, 0.0, u))
    budget = torch.full((1, rows), k, dtype=torch.int32, device=DEV)
    out = (None, None, torch.empty(1, rows, k, dtype=torch.int32, device=DEV), torch.empty(1, rows, dtype=torch.int32, device=DEV))
    took = {}
    for kind, score in kinds.items():
        best = float("inf")
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                ctx.select_gather(score, budget, None, None, w, k, N=P + w, out=out)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 20)
        took[kind] = best
        ref = O.select_indices(score[0, 0].cpu().numpy().astype(np.float64), k, P + w, w)
        assert np.array_equal(out[2][0, 0].cpu().numpy(), ref), kind
    assert max(took.values()) <= 2.0 * took["spread"], took


def test_select_over_workgroups_stale_range_and_small_workspace(ctx):
    from paper_2410_03090_amd import binding
    cfg = synth.tiny_config(dtype="bf16", B=1, H=2, G=2, N=40009, w=32, rank_lo=2, rank_hi=24)
    K, V, Q = synth.gen_all(cfg, seed0=3)
    budget = torch.tensor([[500, 1777]], dtype=torch.int32, device=DEV)
    small = binding.Context(0, 1 << 16)                             # no room to split the rows: one workgroup each
    for change in (None, lambda s: s.copy_(torch.randn(s.shape, device=DEV) * 7), lambda s: s.mul_(1e-6)):
        score = ctx.window_score(Q[0].to(DEV), K[0].to(DEV), G=2, pool=7)
        if change is not None:
            change(score)
        for c in (ctx, ctx, small):                                 # twice: the first call takes the range's place
            _, _, idx, ln = c.select_gather(score, budget, None, None, 32, 1777, N=40009)
            sc = score.cpu().numpy().astype(np.float64)
            for h in range(2):
                ref = O.select_indices(sc[0, h], int(budget[0, h]), 40009, 32)
                assert np.array_equal(idx[0, h, : len(ref)].cpu().numpy(), ref)
    small.close()


# Normalisers folded by the vote workgroups (few partials) and by the merge kernel (many), one and two row groups, rows that
# do not fill the kernel's, one head of many tokens: 1 head has 8 to 128 partials per row here.
@pytest.mark.parametrize("H,G,N,w", [(1, 4, 2100, 32), (1, 4, 16500, 16), (1, 8, 33000, 32), (1, 16, 9000, 32), (1, 2, 140000, 64), (4, 3, 20011, 16)])
def test_score_normalisers_folded(ctx, H, G, N, w):
    cfg = synth.tiny_config(dtype="bf16", B=1, H=H, G=G, N=N, w=w, rank_lo=2, rank_hi=48)
    K, V, Q = synth.gen_all(cfg, seed0=N + G)
    ref = O.window_score(to_f64(Q[0]), to_f64(K[0]), G=G, pool=7)
    np.testing.assert_allclose(ctx.window_score(Q[0].to(DEV), K[0].to(DEV), G=G, pool=7).cpu().numpy(), ref, rtol=2e-5)


# Chunks of the Gram sums: a context with room for the fewest partials only runs and agrees with a larger one to rounding
# (fp32 partial sums in another split: 1e-6), also with the eigen stage beside the scoring kernels.
@pytest.mark.parametrize("dtype,n_mat,N", [("f32", 8, 1024), ("f32", 3, 5000), ("bf16", 8, 4100), ("bf16", 24, 9000)])
def test_entropy_chunks_and_small_workspace(ctx, dtype, n_mat, N):
    from paper_2410_03090_amd import binding
    cfg = synth.tiny_config(dtype=dtype, B=1, H=n_mat, G=2, N=N, w=32, rank_lo=2, rank_hi=48)
    K, V, Q = synth.gen_all(cfg, seed0=N)
    Kd, Qd = K[0].to(DEV), Q[0].to(DEV)
    Href, _ = O.head_entropy(to_f64(K[0, 0]), k_trunc=32)
    least = max(N // 4096, 1)
    chunk = (-(-N // least) + 127) // 128 * 128
    n = -(-N // chunk)
    bytes_least = 32768 + n_mat * n * 128 * 128 * 4 + (n_mat * n * 128 * 4 + 255) // 256 * 256
    score = binding.Context.workspace_bytes(0, N, 128, 1, n_mat, 2, 32) - 32768
    want = ctx.window_score(Qd, Kd, 2, 7)
    for size, overlap in ((bytes_least, False), (bytes_least + score, True), (binding.Context.workspace_bytes(n_mat, N, 128, 1, n_mat, 2, 32), True)):
        c = binding.Context(0, size)
        c.set_overlap(overlap)
        H = c.head_entropy(Kd.view(n_mat, N, 128), k_trunc=32)
        got = c.window_score(Qd, Kd, 2, 7) if overlap else want
        c.join()
        torch.cuda.synchronize()
        np.testing.assert_allclose(H.cpu().numpy(), Href, rtol=1e-5)
        assert torch.equal(got, want)
        c.close()
    np.testing.assert_allclose(ctx.head_entropy(Kd.view(n_mat, N, 128), k_trunc=32).cpu().numpy(), Href, rtol=1e-5)


# Who folds the normalisers: the vote workgroups up to 64 partials a row, up to 16 where a row has one thread (more than 128 query
# rows), the merge kernel beyond.
@pytest.mark.parametrize("G,N,merged", [(4, 16384, False), (8, 8192, False), (8, 10240, True), (8, 16384, True)])
def test_score_who_folds(ctx, G, N, merged):
    cfg = synth.tiny_config(dtype="bf16", B=1, H=1, G=G, N=N, w=32, rank_lo=2, rank_hi=24)
    K, V, Q = synth.gen_all(cfg, seed0=N)
    ctx.profile(True)
    try:
        got = ctx.window_score(Q[0].to(DEV), K[0].to(DEV), G=G, pool=7)
        torch.cuda.synchronize()
        assert ("score_lse" in [name for name, _ in ctx.profile_read()]) == merged
    finally:
        ctx.profile(False)
    np.testing.assert_allclose(got.cpu().numpy(), O.window_score(to_f64(Q[0]), to_f64(K[0]), G=G, pool=7), rtol=2e-5)


# Sums longer than 4096 tokens meet in fp64: tokens 2^11 times larger in the first half of the prompt leave the second half, whose
# products are 2^-32 of the first half's fp32 sums and would vanish there, its own eigenvalue (2^-22 of the trace).  Small whole
# numbers times powers of two: both halves' sums are exact.  1 %: the last bracket of an eigenvalue is 2.9e-10 wide.
@pytest.mark.parametrize("n_mat,N", [(256, 8192), (128, 16384), (300, 8192)])
def test_entropy_halves_of_a_prompt(ctx, n_mat, N):
    v = torch.ones(2, 128)
    v[0, 64:] = -1.0
    X = torch.cat([2048.0 * v[:1].expand(N // 2, 128), v[1:].expand(N // 2, 128)]).to(torch.bfloat16).to(DEV)
    H, eig = ctx.head_entropy(X.expand(n_mat, N, 128), k_trunc=32, flags=0, want_eig=True)
    share = 2.0 ** -22 / (1.0 + 2.0 ** -22)
    want = -share * np.log(share) - (1.0 - share) * np.log1p(-share)
    np.testing.assert_allclose(eig.cpu().numpy()[:, 1], share, rtol=1e-2)
    np.testing.assert_allclose(H.cpu().numpy(), want, rtol=1e-2)


# Layer stages of more layers than a wave and than a workgroup takes at once, of more heads than a wave, against the oracle.
@pytest.mark.parametrize("L,B,H", [(1, 1, 8), (63, 1, 8), (65, 3, 8), (130, 2, 40), (1500, 1, 4), (4096, 1, 2)])
def test_budgets_many_layers(ctx, L, B, H):
    g = torch.Generator().manual_seed(L)
    ent = (3 + torch.rand(L, B, H, generator=g) + torch.cumsum(torch.randn(L, 1, 1, generator=g) * 0.02, 0)).float()
    for flags in (0, 4):
        got = ctx.assign_budgets(ent.to(DEV), H // 2 if H < 8 else 4, 640, 74, 100000, 32, 0.05, 64, flags=flags)
        ref = O.assign_budgets(ent.numpy(), H // 2 if H < 8 else 4, 640, 74, 100000, 32, 0.05, 64, flags=flags)
        for x, y in zip(got, ref):
            assert np.array_equal(x.cpu().numpy(), y)


# Wide bf16 matrices whose rounds run over the covariance (a tile of 256 features a workgroup, 32 tokens a step): token counts
# below a step, with 1 and 31 tokens behind whole steps, several chunks; half and one and a half tiles of features; rows further
# apart than their length; two matrices; with and without the mean.  A context without room for the covariance goes over the tokens.
@pytest.mark.parametrize("N,D,pad", [(20, 256, 0), (33, 384, 8), (700, 640, 0), (2079, 256, 24), (5001, 896, 0), (20000, 512, 8)])
def test_matrix_rounds_over_the_covariance(N, D, pad):
    from paper_2410_03090_amd import binding
    g = torch.Generator().manual_seed(N)
    r = 40
    X = torch.randn(2, N, r, generator=g) @ (torch.randn(r, D, generator=g) * torch.linspace(1.0, 0.05, r)[:, None]) / r
    X = X + 0.01 * torch.randn(2, N, D, generator=g) + 0.2 * torch.randn(D, generator=g)
    X = torch.cat([X, torch.full((2, N, pad), 3.0)], dim=2).to(torch.bfloat16)
    Xd = X.to(DEV)[:, :, :D]
    full = binding.Context.matrix_workspace_bytes(N, D)
    room, tight = binding.Context(0, full), binding.Context(0, full - 4 * D * D)
    try:
        for flags in (O.DEFAULT_FLAGS, O.DEFAULT_FLAGS & ~O.FLAG_CENTER):
            Href, eref = O.head_entropy(to_f64(X[:, :, :D]), k_trunc=32, flags=flags)
            for c, over in ((room, True), (tight, False)):
                c.profile(True)
                H, eig = c.matrix_entropy(Xd, k_trunc=32, n_iter=12, flags=flags, want_eig=True)
                torch.cuda.synchronize()
                assert ("matrix_covariance" in [name for name, _ in c.profile_read()]) == over
                c.profile(False)
                # the final values come from the tokens on either way: the tolerances of the other tests of this call
                np.testing.assert_allclose(H.cpu().numpy(), Href, rtol=1e-4)
                np.testing.assert_allclose(eig.cpu().numpy()[:, :32], eref[:, :32], rtol=0, atol=2e-5)
    finally:
        room.close()
        tight.close()
