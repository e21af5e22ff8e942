"""Parity of the HIP path (through the C ABI) with the CPU oracle on identical seeded inputs.

Tolerances: integer work (union, remap, relabelled targets, statuses) bit-exact; float32
path loss relative error <= 1e-5 and gradient max-abs relative error <= 1e-4; bf16 path
loss relative error <= 2e-3 and gradient cosine >= 0.999 (plus tighter checks that
document the achieved accuracy).
"""
import dataclasses
import functools
import math

import numpy as np
import pytest

import oracle
from paper_2609_33645_amd import workloads
from tests.gpu_util import cosine, loss_rel, rel_err, run_gpu, say, to_dev, unambiguous_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_33645_amd import prunedctc
    prunedctc.lib()  # fails loudly if the HIP library is missing
    yield


# ---------------------------------------------------------------------------------------
# union / remap: bit-exact
# ---------------------------------------------------------------------------------------

@pytest.mark.parametrize("seed,V,blank,Y", [(0, 1000, 0, 17), (1, 180_000, 0, 800), (2, 151_936, 151_935, 650),
                                            (3, 64, 5, 200), (4, 40, 0, 0), (5, 9, 3, 30)])
def test_union_remap_bit_exact(seed, V, blank, Y):
    import torch
    from paper_2609_33645_amd import prunedctc
    say(f"union_remap seed={seed} V={V} blank={blank} Y={Y}")
    rng = np.random.default_rng(seed)
    ids = workloads.zipf_ids(rng, Y, V) if V > 100 else rng.integers(0, V - 1, size=Y).astype(np.int32)
    ids = np.where(ids >= blank, ids + 1, ids).astype(np.int32) if V <= 100 else ids
    ids = np.where(ids == blank, (blank + 1) % V, ids).astype(np.int32)
    ref = oracle.union_remap(ids, [Y], blank, V)
    out = prunedctc.union_remap(torch.from_numpy(ids).cuda(), blank, V)
    assert out["K"] == ref["K"]
    np.testing.assert_array_equal(out["u_ids"].cpu().numpy(), ref["u_ids"])
    np.testing.assert_array_equal(out["remap"].cpu().numpy(), ref["remap"])
    np.testing.assert_array_equal(out["y_rel"].cpu().numpy(), ref["y_rel"])


def test_union_remap_bad_label():
    import torch
    from paper_2609_33645_amd import prunedctc
    with pytest.raises(prunedctc.PrunedCTCError) as e:
        prunedctc.union_remap(torch.tensor([3, 0, 4], dtype=torch.int32, device="cuda"), 0, 10)
    assert e.value.code == -2
    with pytest.raises(prunedctc.PrunedCTCError) as e:
        prunedctc.union_remap(torch.tensor([3, 10], dtype=torch.int32, device="cuda"), 0, 10)
    assert e.value.code == -2


# ---------------------------------------------------------------------------------------
# normaliser and selected log-probabilities
# ---------------------------------------------------------------------------------------

@pytest.mark.parametrize("dtype,M,D,V", [("f32", 92, 64, 1000), ("bf16", 300, 128, 3001), ("bf16", 129, 64, 70_000),
                                         ("f32", 257, 136, 2050), ("bf16", 1, 8, 2), ("bf16", 300, 2056, 5001)])
def test_lse_select(dtype, M, D, V):
    import torch
    from paper_2609_33645_amd import prunedctc
    say(f"lse_select {dtype} M={M} D={D} V={V}")
    rng = np.random.default_rng(M + D + V)
    H = rng.standard_normal((M, D)).astype(np.float32)
    W = (rng.standard_normal((V, D)) / math.sqrt(D)).astype(np.float32) * 3
    if dtype == "bf16":
        H, W = workloads.round_to_bf16(H), workloads.round_to_bf16(W)
    u_ids = np.unique(np.concatenate([[0], rng.integers(1, V, size=min(V - 1, 37))])).astype(np.int32)
    lam_ref = oracle.log_normalizer(H, W, chunk=997)
    S_ref = oracle.selected_logprobs(H, W, u_ids, lam_ref)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    out = prunedctc.lse_select(torch.from_numpy(H).cuda().to(tdt), torch.from_numpy(W).cuda().to(tdt),
                               torch.from_numpy(u_ids).cuda())
    lam = out["lam"].cpu().numpy()
    S = out["S"].cpu().numpy()
    assert np.abs(lam - lam_ref).max() < 2e-5
    assert np.abs(S - S_ref).max() < 5e-5


# ---------------------------------------------------------------------------------------
# alignment stage on seeded scores
# ---------------------------------------------------------------------------------------

def _dp_case(seed, N, Trange, K, U_frac=0.3, p_repeat=0.2, integer=False):
    rng = np.random.default_rng(seed)
    T = rng.integers(Trange[0], Trange[1] + 1, size=N).astype(np.int32)
    U = np.minimum(np.floor(T * U_frac).astype(np.int32), 1023)
    ys = []
    for u in U:
        y = rng.integers(1, K, size=int(u)).astype(np.int32)
        for i in range(1, y.size):
            if rng.random() < p_repeat:
                y[i] = y[i - 1]
        ys.append(y)
    y_rel = np.concatenate(ys) if ys else np.zeros(0, np.int32)
    S = workloads.random_scores(seed + 1000, int(T.sum()), K, integer=integer)
    return S, y_rel, T, U


def _mask_from_margins(res, T, Sp):
    """Expected arc bits (start/stay bit0, step bit1, skip bit2, final bit3) from the
    oracle's fp64 margins."""
    mg = res["margins"]
    want = np.zeros((T, Sp), np.uint8)
    stay = mg["stay"].copy()
    stay[0] = mg["start"]
    want |= (stay >= 0).astype(np.uint8)
    want |= ((mg["step"] >= 0).astype(np.uint8) << 1)
    want |= ((mg["skip"] >= 0).astype(np.uint8) << 2)
    want[T - 1] |= ((mg["final"] >= 0).astype(np.uint8) << 3)
    return want


@pytest.mark.parametrize("seed,N,Trange,K,beam,integer", [
    (0, 3, (1, 40), 20, math.inf, False), (1, 5, (30, 120), 50, math.inf, False),
    (2, 2, (200, 400), 300, math.inf, False), (3, 4, (20, 90), 40, 6.5, True), (4, 3, (50, 150), 64, 12.5, True),
    (5, 2, (300, 500), 200, 16.5, True), (6, 6, (1, 8), 10, 0.5, True), (7, 2, (1500, 1500), 420, 8.5, True),
    (8, 3, (100, 300), 100, math.inf, True), (9, 4, (10, 60), 30, 2.5, True),
    (10, 1, (2100, 2100), 1100, 12.5, True)])  # U = 1023, the longest supported target
def test_ctc_dp_parity(seed, N, Trange, K, beam, integer):
    import torch
    from paper_2609_33645_amd import prunedctc
    S, y_rel, T, U = _dp_case(seed, N, Trange, K, U_frac={7: 0.27, 10: 0.5}.get(seed, 0.3), integer=integer)
    if seed == 10:
        assert U.tolist() == [1023]
    say(f"ctc_dp seed={seed} N={N} T={T.tolist()} U={U.tolist()} K={K} beam={beam}")
    ref = oracle.ctc_from_scores(S.astype(np.float64), y_rel, T, U, beam=beam)
    out = prunedctc.ctc_dp(torch.from_numpy(S).cuda(), torch.from_numpy(y_rel).cuda(), T, U, beam=beam,
                           want_mask=math.isfinite(beam))
    status = out["status"].cpu().numpy()
    np.testing.assert_array_equal(status, ref["status"])
    if math.isfinite(beam):
        # integer scores and a half-integer beam: every margin is >= 0.499 from the threshold,
        # so the kept-arc sets must agree exactly
        mask = out["mask"].cpu().numpy()
        base = 0
        for n in range(N):
            Sp = 2 * int(U[n]) + 1
            mk = mask[base:base + int(T[n]) * Sp].reshape(int(T[n]), Sp)
            base += int(T[n]) * Sp
            if status[n] != 0:
                continue
            fm = ref["per_utt"][n]["margins"]
            finite = [np.abs(v[np.isfinite(v)]) for v in fm.values()]
            assert min((x.min() for x in finite if x.size), default=1.0) > 0.4
            np.testing.assert_array_equal(mk, _mask_from_margins(ref["per_utt"][n], int(T[n]), Sp))
    ln = out["loss_per_utt"].cpu().numpy()
    np.testing.assert_allclose(ln, ref["loss_n"], rtol=2e-6, atol=1e-6)
    G = out["G"].cpu().numpy()
    assert np.abs(G - ref["G"]).max() < 2e-5
    g = out["g"].cpu().numpy()
    assert np.abs(g - ref["g"]).max() < 2e-5


# ---------------------------------------------------------------------------------------
# recomputed backward on identical inputs
# ---------------------------------------------------------------------------------------

@pytest.mark.parametrize("dtype,seed,chunk,D", [("f32", 0, 256, 136), ("bf16", 1, 512, 256), ("bf16", 2, 0, 256),
                                               ("f32", 3, 0, 136), ("bf16", 4, 768, 2056), ("bf16", 5, 0, 2048)])
def test_head_bwd_parity(dtype, seed, chunk, D):
    import torch
    from paper_2609_33645_amd import prunedctc
    wl = workloads.random_small(seed, N=4, T_range=(20, 90) if D < 2048 else (60, 200), D=D, V=3000, dtype=dtype,
                                p_repeat=0.1, beam=5.0, w_std=None if D < 2048 else 0.5 * math.sqrt(128 / D))
    say(f"head_bwd {dtype} seed={seed} M={wl.M} D={wl.D} V={wl.V} chunk={chunk}")
    full = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, 0, beam=wl.beam,
                          want_grads=False)
    ref = oracle.head_backward(wl.H, wl.W, full["lam"], full["G"], full["g"], full["u_ids"])
    H, W, _ = to_dev(wl)
    remap = torch.from_numpy(full["remap"].astype(np.int32)).cuda()
    out = prunedctc.head_bwd(H, W, torch.from_numpy(full["lam"]).cuda(),
                             torch.from_numpy(full["G"].astype(np.float32)).cuda(),
                             torch.from_numpy(full["g"].astype(np.float32)).cuda(), remap, chunk=chunk)
    dH, dW = out["dH"].cpu().numpy(), out["dW"].cpu().numpy()
    if dtype == "f32":
        assert rel_err(dH, ref["dH"]) < 1e-4
        assert rel_err(dW, ref["dW"]) < 1e-4
    else:
        assert cosine(dH, ref["dH"]) > 0.9999
        assert cosine(dW, ref["dW"]) > 0.9999


# ---------------------------------------------------------------------------------------
# end to end
# ---------------------------------------------------------------------------------------

def _check_e2e(wl, res, ref, fp32: bool, tight: bool = True):
    np.testing.assert_array_equal(res["status"], ref["status"])
    lr = loss_rel(res["loss"], ref["loss"])
    say(f"  loss gpu={res['loss']:.9g} oracle={ref['loss']:.9g} rel={lr:.3g}")
    if fp32:
        assert lr <= 1e-5
        assert rel_err(res["dH"], ref["dH"]) <= 1e-4
        assert rel_err(res["dW"], ref["dW"]) <= 1e-4
    else:
        assert lr <= 2e-3
        cH, cW = cosine(res["dH"], ref["dH"]), cosine(res["dW"], ref["dW"])
        say(f"  cos dH={cH:.7f} dW={cW:.7f}")
        assert cH >= 0.999 and cW >= 0.999
        # achieved accuracy is far tighter than the bar: bf16 inputs are exact and only dZ is rounded
        assert lr <= 1e-5
        if tight:
            assert cH >= 0.99999 and cW >= 0.99999


def test_e2e_tiny_f32():
    wl = workloads.tiny_f32(0)
    say(f"e2e tiny_f32 M={wl.M} V={wl.V}")
    ref = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam)
    res = run_gpu(wl)
    _check_e2e(wl, res, ref, fp32=True)


@pytest.mark.parametrize("dtype,D,V,blank", [
    ("bf16", 8, 2, 0), ("f32", 8, 2, 1), ("bf16", 24, 3, 2), ("f32", 24, 1000, 0), ("bf16", 8, 1000, 999),
    ("bf16", 40, 1000, 0), ("bf16", 104, 3001, 5)])
def test_e2e_smallest_shapes(dtype, D, V, blank):
    """The narrowest heads (D = 8, the minimum; D = 24, not a whole k-tile of the products;
    D = 40 and 104, whole k-tiles followed by a partial one, with V = 3001 leaving a partial
    8-column group in the last chunk) and the smallest vocabularies (V = 2: the blank and one
    label), with one-frame utterances among the rest."""
    wl, ref = unambiguous_case(
        lambda s: workloads.random_small(s, N=5, T_range=(1, 5) if V <= 3 else (1, 30), D=D, V=V, dtype=dtype,
                                         token_law="uniform", p_repeat=0.2, blank=blank,
                                         beam=16.0 if V > 3 else math.inf, w_std=0.5), 40 + D + V)
    say(f"e2e smallest {dtype} D={D} V={V} blank={blank} T={wl.input_lengths.tolist()} "
        f"U={wl.target_lengths.tolist()}")
    res = run_gpu(wl)
    # With V <= 3 every class is in the union and dZ = p - gamma is a difference of two O(1)
    # numbers whose dense part p is rounded to bf16: the cancellation amplifies that rounding
    # past the tight check (which assumes p small beside the union columns); the stated bf16
    # tolerance still applies.
    _check_e2e(wl, res, ref, fp32=(dtype == "f32"), tight=V > 3)


@pytest.mark.parametrize("seed,dtype,beam,blank,chunk", [
    (0, "bf16", math.inf, 0, 0), (1, "bf16", 8.0, 0, 512), (2, "f32", math.inf, 7, 256),
    (3, "bf16", 0.0, 0, 0), (4, "f32", 3.0, 2999, 0), (5, "bf16", 16.0, 1500, 1024),
    (6, "bf16", 16.0, 0, 1536),  # two chunks: the second stream's two gated works meet at the last dH
    (7, "f32", 16.0, 0, 1 << 16), (8, "bf16", 16.0, 0, 1 << 16),  # chunk wider than V: one step
    (9, "bf16", 16.0, 0, 256), (10, "bf16", math.inf, 3, 256)])  # one split-K slice: dH accumulated in place
def test_e2e_small(seed, dtype, beam, blank, chunk):
    wl, ref = unambiguous_case(
        lambda s: workloads.random_small(s, N=5, T_range=(1, 140), D=128, V=3000, dtype=dtype, p_repeat=0.15,
                                         blank=blank, beam=beam, w_std=0.5), seed)
    say(f"e2e small seed={seed} {dtype} beam={beam} blank={blank} M={wl.M} T={wl.input_lengths.tolist()}")
    res = run_gpu(wl, chunk=chunk)
    _check_e2e(wl, res, ref, fp32=(dtype == "f32"))


@pytest.mark.parametrize("chunk", [0, 256])
def test_e2e_frozen_head(chunk):
    """A frozen head (dW not requested, the LLM-CTC setting): loss and dH as with dW, from a
    workspace sized for calls without dW; chunk 256 makes the dH product a single split-K slice
    (dH accumulated in place, the union columns' part added after the dense part)."""
    from paper_2609_33645_amd import prunedctc
    wl, ref = unambiguous_case(
        lambda s: workloads.random_small(s, N=5, T_range=(20, 140), D=256, V=4000, dtype="bf16", p_repeat=0.1,
                                         beam=16.0, w_std=0.5 * math.sqrt(128 / 256)), 70 + chunk)
    say(f"e2e frozen head chunk={chunk} M={wl.M}")
    res = run_gpu(wl, chunk=chunk, want_dW=False)
    assert res["workspace_bytes"] == prunedctc.workspace_size(1, wl.input_lengths, wl.target_lengths, wl.D, wl.V,
                                                              wl.beam, chunk, want_dW=False)
    assert res["workspace_bytes"] < prunedctc.workspace_size(1, wl.input_lengths, wl.target_lengths, wl.D, wl.V,
                                                             wl.beam, chunk)
    np.testing.assert_array_equal(res["status"], ref["status"])
    assert loss_rel(res["loss"], ref["loss"]) <= 1e-5
    assert cosine(res["dH"], ref["dH"]) >= 0.99999


def test_e2e_edge_cases():
    """Empty target, unalignable utterance, NaN in H, all classes selected (K = V)."""
    import torch
    rng = np.random.default_rng(9)
    V, D = 16, 32
    T = np.array([6, 2, 9, 5, 7], np.int32)
    U = np.array([0, 2, 3, 2, 15], np.int32)
    U[4] = 6
    ys = [np.zeros(0, np.int32), np.array([4, 4], np.int32), np.array([1, 2, 3], np.int32),
          np.array([5, 6], np.int32), np.arange(10, 16, dtype=np.int32)]
    targets = np.concatenate(ys)
    H = workloads.round_to_bf16(rng.standard_normal((int(T.sum()), D)).astype(np.float32))
    W = workloads.round_to_bf16(rng.standard_normal((V, D)).astype(np.float32) * 0.3)
    H[6 + 2 + 9 + 1, 3] = np.nan           # utterance 3 gets a NaN frame
    wl = workloads.Workload("edge", "bf16", H, W, targets, T, U, 0, math.inf)
    ref = oracle.fwd_bwd(H, W, targets, T, U, 0)
    assert ref["status"].tolist() == [0, 1, 0, 2, 0]
    res = run_gpu(wl)
    np.testing.assert_array_equal(res["status"], ref["status"])
    assert np.isfinite(res["dW"]).all() and np.isfinite(res["dH"]).all()
    assert loss_rel(res["loss"], ref["loss"]) < 1e-5
    assert cosine(res["dW"], ref["dW"]) > 0.99999
    assert cosine(res["dH"], ref["dH"]) > 0.99999
    # all classes selected: every id in [0, V) occurs
    H2 = workloads.round_to_bf16(rng.standard_normal((40, D)).astype(np.float32))
    wl2 = workloads.Workload("allsel", "bf16", H2, W, np.arange(1, 16, dtype=np.int32), np.array([40], np.int32),
                             np.array([15], np.int32), 0, math.inf)
    ref2 = oracle.fwd_bwd(H2, W, wl2.targets, wl2.input_lengths, wl2.target_lengths, 0)
    assert ref2["K"] == V
    res2 = run_gpu(wl2)
    assert loss_rel(res2["loss"], ref2["loss"]) < 1e-5
    assert cosine(res2["dW"], ref2["dW"]) > 0.99999
    assert cosine(res2["dH"], ref2["dH"]) > 0.99999
    del torch


@pytest.mark.parametrize("seed,N,Trange,V,u_frac", [
    (61, 1000, (1, 12), 2000, 0.25),        # many short utterances (one lattice wavefront pair each)
    (62, 1, (40000, 40000), 1000, 0.0025)])  # one very long utterance (40,000 sequential frames)
def test_e2e_batch_extremes(seed, N, Trange, V, u_frac):
    wl, ref = unambiguous_case(
        lambda s: workloads.random_small(s, N=N, T_range=Trange, D=64, V=V, dtype="bf16", p_repeat=0.1,
                                         u_frac=u_frac, beam=16.0, w_std=0.5), seed)
    say(f"e2e batch extremes N={N} M={wl.M} U_total={int(wl.target_lengths.sum())}")
    res = run_gpu(wl)
    _check_e2e(wl, res, ref, fp32=False)


def test_e2e_max_vocab():
    """The largest supported vocabulary (524,288 classes: the limit of the union's on-chip
    membership bitmap) with the blank at the last id, labels drawn over the whole range, and
    several backward chunks."""
    V = 524288
    wl, ref = unambiguous_case(
        lambda s: workloads.random_small(s, N=3, T_range=(20, 60), D=64, V=V, dtype="bf16", token_law="uniform",
                                         p_repeat=0.1, blank=V - 1, beam=16.0, w_std=0.5), 12)
    say(f"e2e max vocabulary V={V} M={wl.M} T={wl.input_lengths.tolist()}")
    res = run_gpu(wl, chunk=65536)
    _check_e2e(wl, res, ref, fp32=False)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_e2e_empty_batch(dtype):
    """No utterances (N = 0, M = 0): the loss is an empty sum (0), every head-gradient entry
    is 0 (dW and db are written, not left as they were), and the call succeeds."""
    import torch
    from paper_2609_33645_amd import prunedctc
    say(f"empty batch {dtype}")
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    V, D = 300, 64
    gen = torch.Generator(device="cpu").manual_seed(5)
    H = torch.zeros((0, D), dtype=tdt, device="cuda")
    W = torch.randn((V, D), generator=gen).to(tdt).cuda()
    targets = torch.zeros(0, dtype=torch.int32, device="cuda")
    bias = torch.randn(V, generator=gen).cuda()
    for kw in ({}, {"bias": bias, "want_db": True}):
        dW_out = torch.full((V, D), float("nan"), device="cuda")
        res = prunedctc.pruned_ctc_fwd_bwd(H, W, targets, [], [], 0, 16.0, dW_out=dW_out, **kw)
        torch.cuda.synchronize()
        assert res["loss"].item() == 0.0
        assert res["dH"].shape == (0, D) and res["loss_per_utt"].numel() == 0
        assert torch.count_nonzero(torch.nan_to_num(res["dW"], nan=1.0)).item() == 0
        if kw:
            assert torch.count_nonzero(res["db"]).item() == 0


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_stage_entry_points_without_frames(dtype):
    """Each stage entry point accepts a batch without frames: nothing to compute, no error,
    and the head gradient of an empty sum is written as zeros."""
    import torch
    from paper_2609_33645_amd import prunedctc
    say(f"stages without frames {dtype}")
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    V, D, K = 300, 64, 3
    gen = torch.Generator(device="cpu").manual_seed(6)
    H = torch.zeros((0, D), dtype=tdt, device="cuda")
    W = torch.randn((V, D), generator=gen).to(tdt).cuda()
    u_ids = torch.tensor([0, 5, 9], dtype=torch.int32, device="cuda")
    sel = prunedctc.lse_select(H, W, u_ids)
    assert sel["lam"].numel() == 0
    S = torch.zeros((0, K), dtype=torch.float32, device="cuda")
    y_rel = torch.zeros(0, dtype=torch.int32, device="cuda")
    dp = prunedctc.ctc_dp(S, y_rel, [], [], 16.0)
    assert dp["loss_per_utt"].numel() == 0
    dec = prunedctc.greedy_decode(H, W, [], 0)
    assert dec["tokens"] == []
    assert prunedctc.discarded_mass(S, y_rel, [], [], [1.0, 16.0]).numel() == 0
    remap = torch.full((V,), -1, dtype=torch.int32, device="cuda")
    bwd = prunedctc.head_bwd(H, W, torch.zeros(0, dtype=torch.float64, device="cuda"), S,
                             torch.zeros(0, dtype=torch.float32, device="cuda"), remap)
    torch.cuda.synchronize()
    assert bwd["dH"].shape == (0, D) and torch.count_nonzero(bwd["dW"]).item() == 0
    gl = prunedctc.grouped_logprobs(H, W, u_ids)
    assert gl["logp"].shape == (0, K + 1) and gl["lam"].numel() == 0


@pytest.mark.parametrize("beam", [math.inf, 0.0])
def test_e2e_tight_alignment(beam):
    """Utterances whose targets fill their frames exactly (T = U + repeats) have one alignment
    (the labels, with a blank only between equal neighbours): the loss is minus the sum of its
    log-probabilities (fp64 closed form here), pruned or not."""
    rng = np.random.default_rng(77)
    V, D = 500, 64
    ys = [np.array([3, 3, 7], np.int32), np.array([9], np.int32), np.array([4, 5, 5, 5, 6], np.int32)]
    paths = []
    for y in ys:
        pth, prev = [], None
        for c in y.tolist():
            if c == prev:
                pth.append(0)  # the blank (id 0) between equal neighbours
            pth.append(c)
            prev = c
        paths.append(pth)
    T = np.array([len(q) for q in paths], np.int32)
    U = np.array([len(y) for y in ys], np.int32)
    H = workloads.round_to_bf16(rng.standard_normal((int(T.sum()), D)).astype(np.float32))
    W = workloads.round_to_bf16(rng.standard_normal((V, D)).astype(np.float32) * 0.3)
    wl = workloads.Workload("tight", "bf16", H, W, np.concatenate(ys), T, U, 0, beam)
    say(f"e2e tight alignment beam={beam} T={T.tolist()} U={U.tolist()}")
    z = H.astype(np.float64) @ W.astype(np.float64).T
    zmax = z.max(axis=1, keepdims=True)
    logp = z - (zmax + np.log(np.exp(z - zmax).sum(axis=1, keepdims=True)))
    path = np.concatenate([np.asarray(q) for q in paths])
    want = -logp[np.arange(path.size), path].sum()
    res = run_gpu(wl)
    assert res["status"].tolist() == [0, 0, 0]
    assert abs(res["loss"] - want) <= 1e-5 * abs(want)
    ref = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam)
    _check_e2e(wl, res, ref, fp32=False)


# Both schedules of the second stream (pctc_lattice_leads): the least vocabulary that 64 utterances
# of 20 frames have their lattice gated at, and one class fewer, where it runs ungated.
_SCHED_T = np.full(64, 20, np.int32)
_SCHED_U = np.full(64, 4, np.int32)
_SCHED_D, _SCHED_BEAM = 512, 16.0


@functools.lru_cache(maxsize=None)
def _gated_from():
    from paper_2609_33645_amd import prunedctc
    lo, hi = 2, 400_000  # leads at lo, gated at hi
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lead = prunedctc.lattice_leads(prunedctc.PCTC_BF16, _SCHED_T, _SCHED_U, _SCHED_D, mid, _SCHED_BEAM)
        lo, hi = (mid, hi) if lead else (lo, mid)
    return hi


@functools.lru_cache(maxsize=None)
def _schedule_case(gated, bias):
    """(workload, bias, oracle's result).  "miss": one target's bias is -inf, "nan": a frame is not a
    number; the forecast of that utterance is wrong and the backward done again in the plain order."""
    V = _gated_from() - (0 if gated else 1)
    wl = workloads.synthesize(name="sched", dtype="bf16", T=_SCHED_T, U=_SCHED_U, D=_SCHED_D, V=V, beam=_SCHED_BEAM,
                              rng=np.random.default_rng(20))
    b = None
    if bias == "nan":
        wl.H[25, 3] = np.nan  # a frame of the second utterance
    elif bias:
        b = np.random.default_rng(21).standard_normal(V).astype(np.float32) * 0.5
        if bias == "miss":
            b[int(wl.targets[5])] = -np.inf
    ref = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam, bias=b)
    return wl, b, ref


@pytest.mark.parametrize("gated", [True, False])
@pytest.mark.parametrize("chunk,outputs,bias", [
    (0, "dH dW", None), (65_536, "dH dW", None),   # one chunk
    (32_768, "dH dW", None), (32_768, "dH", None), (32_768, "dW", None),
    (16_384, "dH dW", None), (16_384, "dH", None), (16_384, "dW", None),
    (256, "dH dW", None), (256, "dH", None),       # dH in one slice: summed in place
    (16_384, "dH dW db", "plain"), (65_536, "dH dW db", "plain"), (16_384, "db", "plain"),
    (16_384, "dH dW db", "miss"), (256, "dH dW db", "miss"), (0, "dH dW", "nan"), (256, "dH dW", "nan"),
])
def test_e2e_lattice_schedules(gated, chunk, outputs, bias):
    """Gated and ungated lattice beside the dense part, on both sides of the rule's edge: one, two and
    more chunks, dH in slices and in place, a frozen head, dW or db alone, and a wrong forecast."""
    import torch
    from paper_2609_33645_amd import prunedctc
    wl, b, ref = _schedule_case(gated, bias)
    assert prunedctc.lattice_leads(prunedctc.PCTC_BF16, wl.input_lengths, wl.target_lengths, wl.D, wl.V,
                                   wl.beam) == (not gated)
    assert prunedctc.bwd_chunk(prunedctc.PCTC_BF16, wl.M, wl.D, wl.V, 65_536) >= wl.V
    say(f"lattice schedules gated={gated} V={wl.V} chunk={chunk} {outputs} bias={bias}")
    H, W, y = to_dev(wl)
    out = prunedctc.pruned_ctc_fwd_bwd(H, W, y, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam, chunk=chunk,
                                       want_dH="dH" in outputs, want_dW="dW" in outputs, want_db="db" in outputs,
                                       bias=None if b is None else torch.from_numpy(b).cuda())
    np.testing.assert_array_equal(out["status"].cpu().numpy(), ref["status"])
    assert (ref["status"] != 0).any() == (bias in ("miss", "nan"))
    assert loss_rel(float(out["loss"].item()), ref["loss"]) <= 1e-5
    for name in outputs.split():
        got = out[name].cpu().numpy()
        assert np.isfinite(got).all(), name
        assert cosine(got, ref[name]) >= 0.99999, name


@pytest.mark.parametrize("nthreads", [2, 6])
def test_concurrent_calls_on_streams(nthreads):
    """Host threads, each on its own stream with its own workspace and outputs, run the fused
    call at the same time (each caller stream has its own second stream, up to four per
    device; with six, some share one): every result equals that of the same call made
    alone, bit for bit."""
    import threading
    import torch
    from paper_2609_33645_amd import prunedctc
    say(f"concurrent calls on {nthreads} streams")
    wls = [workloads.random_small(90 + i, N=6, T_range=(40, 160), D=128, V=3000, dtype="bf16", p_repeat=0.1,
                                  beam=16.0, w_std=0.5) for i in range(nthreads)]

    def call(wl):
        H, W, y = to_dev(wl)
        out = prunedctc.pruned_ctc_fwd_bwd(H, W, y, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam)
        torch.cuda.current_stream().synchronize()
        return [out["loss"].cpu(), out["status"].cpu(), out["dH"].cpu(), out["dW"].cpu()]

    alone = [call(wl) for wl in wls]
    results = [[None] * 3 for _ in wls]
    errors = []

    def worker(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for r in range(3):
                    results[i][r] = call(wls[i])
        except Exception as e:  # reported below
            errors.append(repr(e))

    threads = [threading.Thread(target=worker, args=(i,)) for i in range(nthreads)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
    assert not any(t.is_alive() for t in threads)
    assert not errors, errors
    for i in range(nthreads):
        for r in range(3):
            for a, b in zip(results[i][r], alone[i]):
                assert torch.equal(a, b), (i, r)


def test_error_codes():
    import torch
    from paper_2609_33645_amd import prunedctc
    H = torch.zeros((5, 8), dtype=torch.bfloat16, device="cuda")
    W = torch.zeros((10, 8), dtype=torch.bfloat16, device="cuda")
    y = torch.tensor([1, 2], dtype=torch.int32, device="cuda")
    for targets, T, U, blank, beam, code in [
        ([1, 0], [2, 3], [1, 1], 0, math.inf, -2),    # label == blank (device check)
        ([1, 12], [2, 3], [1, 1], 0, math.inf, -2),   # label out of range (device check)
        ([1, 2], [0, 5], [1, 1], 0, math.inf, -3),    # T_n < 1
        ([1, 2], [2, 3], [1, 1], 10, math.inf, -1),   # blank out of range
        ([1, 2], [2, 3], [1, 1], 0, float("nan"), -1),
    ]:
        with pytest.raises(prunedctc.PrunedCTCError) as e:
            prunedctc.pruned_ctc_fwd_bwd(H, W, torch.tensor(targets, dtype=torch.int32, device="cuda"), T, U,
                                         blank, beam)
        assert e.value.code == code, (targets, T, U, blank, beam)
    del y


# ---------------------------------------------------------------------------------------
# head bias, blank offset, loss weights and the bias gradient (pruned_ctc_fwd_bwd_ex)
# ---------------------------------------------------------------------------------------

@pytest.mark.parametrize("seed,dtype,beam,blank,chunk,zero_w,D", [
    (0, "f32", math.inf, 0, 256, False, 128), (1, "bf16", 16.0, 0, 0, True, 128),
    (2, "bf16", math.inf, 2999, 512, False, 128), (3, "f32", 4.0, 11, 0, True, 128),
    (4, "bf16", 0.0, 0, 1024, False, 128), (5, "bf16", 16.0, 3, 0, False, 2056),
    (6, "bf16", 16.0, 0, 256, True, 128)])  # dH accumulated in place, union part added after it
def test_e2e_bias_weights_db(seed, dtype, beam, blank, chunk, zero_w, D):
    import torch
    from paper_2609_33645_amd import prunedctc
    rng = np.random.default_rng(seed)
    b = rng.standard_normal(3000).astype(np.float32)
    b[blank] += 2.0                                  # blank offset eta
    w = rng.uniform(0.05, 2.0, size=5).astype(np.float32)
    if zero_w:
        w[1] = 0.0
    wl, ref = unambiguous_case(
        lambda s: workloads.random_small(s, N=5, T_range=(1, 140), D=D, V=3000, dtype=dtype, p_repeat=0.15,
                                         blank=blank, beam=beam, w_std=0.5 * math.sqrt(128 / D)), 40 + seed,
        bias=b.astype(np.float64), weights=w.astype(np.float64))
    say(f"e2e bias/weights seed={seed} {dtype} beam={beam} blank={blank} M={wl.M} w={np.round(w, 3).tolist()}")
    H, W, y = to_dev(wl)
    out = prunedctc.pruned_ctc_fwd_bwd(H, W, y, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam, chunk=chunk,
                                       bias=torch.from_numpy(b).cuda(), utt_weight=torch.from_numpy(w).cuda(),
                                       want_db=True)
    res = {"loss": float(out["loss"].item()), "status": out["status"].cpu().numpy(), "dH": out["dH"].cpu().numpy(),
           "dW": out["dW"].cpu().numpy()}
    np.testing.assert_allclose(out["loss_per_utt"].cpu().numpy(), ref["loss_n"], rtol=1e-5, atol=1e-6)
    _check_e2e(wl, res, ref, fp32=(dtype == "f32"))
    db = out["db"].cpu().numpy()
    cdb = cosine(db, ref["db"])
    say(f"  db cos={cdb:.7f} rel={rel_err(db, ref['db']):.3g}  d_eta gpu={db[blank]:.6g} oracle={ref['db'][blank]:.6g}")
    if dtype == "f32":
        assert rel_err(db, ref["db"]) <= 1e-4
    else:
        assert cdb >= 0.999
        assert cdb >= 0.99999
    assert abs(db[blank] - ref["db"][blank]) <= 2e-3 * max(1.0, abs(ref["db"][blank]))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_e2e_negative_weights(dtype):
    """Loss weights of either sign (and a zero): g = -w_n changes sign with the weight, and only
    a zero weight removes an utterance from the backward."""
    import torch
    from paper_2609_33645_amd import prunedctc
    w = np.array([1.5, -0.4, 0.0, -0.6, 1.2], np.float32)
    b = np.random.default_rng(57).standard_normal(3000).astype(np.float32)
    wl, ref = unambiguous_case(
        lambda s: workloads.random_small(s, N=5, T_range=(20, 140), D=128, V=3000, dtype=dtype, p_repeat=0.15,
                                         beam=16.0, w_std=0.5), 57,
        bias=b.astype(np.float64), weights=w.astype(np.float64))
    say(f"e2e negative weights {dtype} M={wl.M} w={w.tolist()}")
    H, W, y = to_dev(wl)
    out = prunedctc.pruned_ctc_fwd_bwd(H, W, y, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam,
                                       bias=torch.from_numpy(b).cuda(), utt_weight=torch.from_numpy(w).cuda(),
                                       want_db=True)
    res = {"loss": float(out["loss"].item()), "status": out["status"].cpu().numpy(), "dH": out["dH"].cpu().numpy(),
           "dW": out["dW"].cpu().numpy()}
    np.testing.assert_allclose(out["loss_per_utt"].cpu().numpy(), ref["loss_n"], rtol=1e-5, atol=1e-6)
    _check_e2e(wl, res, ref, fp32=(dtype == "f32"))
    db = out["db"].cpu().numpy()
    if dtype == "f32":
        assert rel_err(db, ref["db"]) <= 1e-4
    else:
        assert cosine(db, ref["db"]) >= 0.99999


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_e2e_masked_vocabulary(dtype):
    """A -inf bias on many non-target classes (a masked vocabulary, including whole runs of
    normaliser tiles): those classes get probability 0, so zero gradient rows in dW and db."""
    import torch
    from paper_2609_33645_amd import prunedctc
    def masked_bias(wl):
        rng = np.random.default_rng(58)
        b = rng.standard_normal(wl.V).astype(np.float32)
        masked = rng.random(wl.V) < 0.3
        masked[2048:3072] = True                      # whole tiles with no finite logit
        masked[np.unique(wl.targets)] = False
        masked[wl.blank] = False
        b[masked] = -np.inf
        return b, masked

    wl, ref = unambiguous_case(
        lambda s: workloads.random_small(s, N=4, T_range=(20, 120), D=128, V=5000, dtype=dtype, p_repeat=0.15,
                                         beam=16.0, w_std=0.5), 58,
        kw_of=lambda wl: {"bias": masked_bias(wl)[0].astype(np.float64)})
    b, masked = masked_bias(wl)
    say(f"e2e masked vocabulary {dtype} M={wl.M} masked={int(masked.sum())}")
    H, W, y = to_dev(wl)
    out = prunedctc.pruned_ctc_fwd_bwd(H, W, y, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam,
                                       bias=torch.from_numpy(b).cuda(), want_db=True)
    res = {"loss": float(out["loss"].item()), "status": out["status"].cpu().numpy(), "dH": out["dH"].cpu().numpy(),
           "dW": out["dW"].cpu().numpy()}
    _check_e2e(wl, res, ref, fp32=(dtype == "f32"))
    db = out["db"].cpu().numpy()
    assert np.all(db[masked] == 0.0) and np.all(res["dW"][masked] == 0.0)
    assert np.isfinite(db).all() and np.isfinite(res["dW"]).all() and np.isfinite(res["dH"]).all()


@pytest.mark.parametrize("dtype,beam", [("bf16", 16.0), ("f32", math.inf)])
def test_e2e_large_logits(dtype, beam):
    """Logits with a spread of hundreds of nats (near one-hot probabilities: the exponentials
    underflow for almost every class, the lattice's scores move by hundreds per frame)."""
    wl, ref = unambiguous_case(
        lambda s: workloads.random_small(s, N=4, T_range=(20, 120), D=128, V=3000, dtype=dtype, p_repeat=0.15,
                                         beam=beam, w_std=5.0), 59)
    say(f"e2e large logits {dtype} beam={beam} M={wl.M}")
    res = run_gpu(wl)
    _check_e2e(wl, res, ref, fp32=(dtype == "f32"))


@pytest.mark.parametrize("case", ["in_range", "high", "low"])
def test_e2e_first_chunk_from_normaliser(case):
    """Narrow bf16 heads: the normaliser writes the first backward chunk's rows as exp(z) and
    the backward applies each frame's factor -g exp(-lambda) afterwards (Eq. vjp; no recompute
    of that chunk).  That is usable while every lambda lies in [-40, 60]; frames whose lambda
    leaves that range (high: logits scaled up; low: every logit far below zero) make the
    call recompute the chunk instead.  Each case is checked against the oracle with the
    default chunk (two chunks, the first from the normaliser when usable) and with an explicit
    chunk that is not a whole number of normaliser partitions (every chunk recomputed)."""
    wl = workloads.random_small(7, N=4, T_range=(40, 90), D=128, V=70_000, dtype="bf16")
    if case != "in_range":
        H, W = wl.H.copy(), wl.W.copy()
        if case == "high":
            H[:10] *= 20.0  # logits of those frames scaled by 20: lambda up to about 100
        else:
            u = np.full(wl.D, 1.0 / np.sqrt(wl.D), np.float32)
            W = W + u  # a common direction in every class row
            H[:10] = -100.0 * u  # those frames: every logit near -100, lambda about -60
        wl = dataclasses.replace(wl, H=workloads.round_to_bf16(H), W=workloads.round_to_bf16(W))
    ref = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam)
    lam = ref["lam"]
    say(f"e2e first chunk from the normaliser: {case} M={wl.M} lambda in [{lam.min():.1f}, {lam.max():.1f}]")
    if case == "in_range":
        assert lam.min() >= -40 and lam.max() <= 60
    else:
        assert lam.min() < -40 or lam.max() > 60
    for chunk in (0, 36608):
        res = run_gpu(wl, chunk=chunk)
        say(f"  chunk {chunk}")
        _check_e2e(wl, res, ref, fp32=False)


# ---------------------------------------------------------------------------------------
# discarded posterior mass (App. B.3)
# ---------------------------------------------------------------------------------------

@pytest.mark.parametrize("seed,N,Trange,K", [(0, 4, (20, 90), 40), (1, 3, (100, 300), 120), (2, 2, (1500, 1500), 420)])
def test_discarded_mass(seed, N, Trange, K):
    import torch
    from paper_2609_33645_amd import prunedctc
    # integer scores and half-integer beams: every arc decision is at least 0.499 from the
    # threshold, so both sides retain the same arcs
    S, y_rel, T, U = _dp_case(60 + seed, N, Trange, K, U_frac=0.27 if seed == 2 else 0.3, integer=True)
    beams = [0.5, 2.5, 6.5, 12.5, 30.5, 1.0e4]
    say(f"discarded mass seed={seed} N={N} T={T.tolist()} U={U.tolist()} beams={beams}")
    ref = oracle.discarded_mass(S.astype(np.float64), y_rel, T, U, beams)
    got = prunedctc.discarded_mass(torch.from_numpy(S).cuda(), torch.from_numpy(y_rel).cuda(), T, U, beams)
    got = got.cpu().numpy()
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    ok = ~np.isnan(ref)
    err = np.abs(got[ok] - ref[ok])
    say(f"  max delta {np.nanmax(ref):.3g}; max |gpu - oracle| {err.max() if err.size else 0:.3g}")
    assert np.all(err <= 1e-10 + 1e-5 * np.abs(ref[ok]))
    assert np.all(got[-1][ok[-1]] == 0.0)  # a beam above every margin drops nothing


def test_beam_sweep_tool():
    """The sweep tool end to end on a small bf16 batch: deltas agree with the oracle's on the
    same S (the oracle's S), decrease with the beam, and the required beam is the first beam
    whose maximum is within the criterion."""
    import torch
    from paper_2609_33645_amd import beam_sweep
    wl = workloads.random_small(77, N=4, T_range=(30, 120), D=64, V=2000, dtype="bf16", p_repeat=0.1, w_std=0.4)
    H, W, y = to_dev(wl)
    beams = [2.0, 8.0, 32.0, 200.0]
    res = beam_sweep.beam_sweep(H, W, y, wl.input_lengths, wl.target_lengths, wl.blank, beams)
    mx = [r["max_delta"] for r in res["rows"]]
    say(f"beam sweep: {[(r['beam'], r['max_delta'], r['above']) for r in res['rows']]} required={res['required_beam']}")
    assert all(mx[i] >= mx[i + 1] - 1e-12 for i in range(len(mx) - 1))
    first_ok = next((r["beam"] for r in res["rows"] if r["above"] == 0), None)
    assert res["required_beam"] == first_ok
    ref = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, wl.blank, math.inf,
                         want_grads=False)
    d_ref = oracle.discarded_mass(ref["S"], ref["y_rel"], wl.input_lengths, wl.target_lengths, beams)
    # float scores on both sides: compare where the oracle's delta is well above rounding
    big = d_ref > 1e-6
    np.testing.assert_allclose(res["delta"][big], d_ref[big], rtol=2e-3)


# ---------------------------------------------------------------------------------------
# greedy emission head
# ---------------------------------------------------------------------------------------

def _check_greedy(wl, H64, W64, b64, got, ref, frames=None, eps=1e-3):
    """ids agree wherever the oracle's best logit leads the runner-up by more than eps; at
    nearer ties the GPU's id must score within eps of the best.  Token sequences agree for
    utterances without near ties and are always the collapse of the GPU's own ids."""
    ids = got["ids"].cpu().numpy()
    if frames is not None:
        ids = ids[frames]
    sure = (ref["best"] - ref["second"]) > eps
    np.testing.assert_array_equal(ids[sure], ref["ids"][sure])
    rows = np.nonzero(~sure)[0]
    fr = rows if frames is None else frames[rows]
    if rows.size:
        z = np.einsum("md,md->m", H64[fr], W64[ids[rows]]) + b64[ids[rows]]
        assert np.all(z >= ref["best"][rows] - eps)
    say(f"  greedy: {int(sure.sum())} frames decided, {rows.size} near ties")
    return ids, sure


@pytest.mark.parametrize("seed,dtype,blank,with_bias,D", [(0, "f32", 0, False, 128), (1, "bf16", 0, True, 128),
                                                          (2, "bf16", 2999, False, 128), (3, "f32", 5, True, 128),
                                                          (4, "bf16", 7, True, 2056), (5, "bf16", 0, False, 2048)])
def test_greedy_decode(seed, dtype, blank, with_bias, D):
    import torch
    from paper_2609_33645_amd import prunedctc
    wl = workloads.random_small(90 + seed, N=6, T_range=(1, 150), D=D, V=3000, dtype=dtype, blank=blank,
                                w_std=0.5 * math.sqrt(128 / D))
    H, W, _ = to_dev(wl)
    rng = np.random.default_rng(seed)
    b = rng.standard_normal(wl.V).astype(np.float32) if with_bias else np.zeros(wl.V, np.float32)
    # a duplicated class row makes exact ties, broken toward the smaller id
    Wn = wl.W.copy()
    Wn[2500] = Wn[33]
    b[2500] = b[33]
    W = torch.from_numpy(Wn).cuda().to(H.dtype)
    say(f"greedy seed={seed} {dtype} blank={blank} bias={with_bias} M={wl.M} T={wl.input_lengths.tolist()}")
    got = prunedctc.greedy_decode(H, W, wl.input_lengths, blank, bias=torch.from_numpy(b).cuda() if with_bias else None)
    H64, W64, b64 = wl.H.astype(np.float64), Wn.astype(np.float64), b.astype(np.float64)
    ref = oracle.greedy_decode(H64, W64, wl.input_lengths, blank, bias=b64)
    ids, sure = _check_greedy(wl, H64, W64, b64, got, ref)
    assert not np.any(ids == 2500)
    off = np.concatenate([[0], np.cumsum(wl.input_lengths)])
    for n in range(wl.N):
        own = oracle.ctc_collapse(ids[off[n]:off[n + 1]], blank)
        assert got["tokens"][n] == own
        if sure[off[n]:off[n + 1]].all():
            assert got["tokens"][n] == ref["tokens"][n]


@pytest.mark.parametrize("dtype,D,V,blank", [("f32", 8, 2, 0), ("bf16", 8, 2, 1), ("bf16", 24, 3, 2),
                                               ("f32", 24, 300, 299)])
def test_greedy_decode_smallest_shapes(dtype, D, V, blank):
    """The greedy head at the narrowest widths and the smallest vocabularies, with one-frame
    utterances."""
    import torch
    from paper_2609_33645_amd import prunedctc
    wl = workloads.random_small(70 + D + V, N=5, T_range=(1, 9), D=D, V=V, dtype=dtype, blank=blank, w_std=0.5)
    H, W, _ = to_dev(wl)
    say(f"greedy smallest {dtype} D={D} V={V} T={wl.input_lengths.tolist()}")
    got = prunedctc.greedy_decode(H, W, wl.input_lengths, blank)
    H64, W64, b64 = wl.H.astype(np.float64), wl.W.astype(np.float64), np.zeros(V)
    ref = oracle.greedy_decode(H64, W64, wl.input_lengths, blank, bias=b64)
    ids, sure = _check_greedy(wl, H64, W64, b64, got, ref)
    off = np.concatenate([[0], np.cumsum(wl.input_lengths)])
    for n in range(wl.N):
        assert got["tokens"][n] == oracle.ctc_collapse(ids[off[n]:off[n + 1]], blank)
        if sure[off[n]:off[n + 1]].all():
            assert got["tokens"][n] == ref["tokens"][n]


# ---------------------------------------------------------------------------------------
# grouped logits for a stock CTC (Eq. grouped, Prop. 1, Eq. offsupport)
# ---------------------------------------------------------------------------------------

def _stock_ctc(torch, logp, y_rel, T, U, dev):
    """torch's own CTC over K + 1 classes (blank = column 0) on [M, K + 1] log-probabilities."""
    off = np.concatenate([[0], np.cumsum(T)])
    Tm = int(T.max())
    pad = torch.stack([torch.nn.functional.pad(logp[off[n]:off[n + 1]], (0, 0, 0, Tm - int(T[n])))
                       for n in range(len(T))], 1)
    return torch.nn.functional.ctc_loss(pad, torch.as_tensor(y_rel, dtype=torch.long, device=dev),
                                        torch.as_tensor(T, dtype=torch.long), torch.as_tensor(U, dtype=torch.long),
                                        blank=0, reduction="sum")


@pytest.mark.parametrize("seed,dtype,with_bias,chunk", [(0, "f32", False, 0), (1, "bf16", True, 512),
                                                        (2, "bf16", False, 0), (3, "f32", True, 256)])
def test_grouped_export(seed, dtype, with_bias, chunk):
    """Export vs the oracle element by element; then torch's CTC on the GPU over the export,
    through the autograd wrapper, against the full-vocabulary loss and gradients (Prop. 1)."""
    import torch
    from paper_2609_33645_amd import prunedctc
    wl = workloads.random_small(60 + seed, N=4, T_range=(20, 150), D=128, V=3000, dtype=dtype, p_repeat=0.15,
                                w_std=0.5)
    rng = np.random.default_rng(seed)
    b = rng.standard_normal(wl.V).astype(np.float32) if with_bias else None
    b64 = None if b is None else b.astype(np.float64)
    u = oracle.union_remap(wl.targets, wl.target_lengths, wl.blank, wl.V)
    say(f"grouped seed={seed} {dtype} bias={with_bias} chunk={chunk} M={wl.M} K={u['K']} "
        f"T={wl.input_lengths.tolist()}")
    ex = oracle.grouped_logprobs(wl.H, wl.W, u["u_ids"], bias=b64)
    full = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, wl.blank, bias=b64)
    H, W, _ = to_dev(wl)
    uid = torch.from_numpy(u["u_ids"].astype(np.int32)).cuda()
    bt = None if b is None else torch.from_numpy(b).cuda()
    out = prunedctc.grouped_logprobs(H, W, uid, bias=bt)
    logp = out["logp"].cpu().numpy()
    assert logp.shape == ex["logp"].shape
    say(f"  logp max err {np.abs(logp - ex['logp']).max():.3g}  lam max err "
        f"{np.abs(out['lam'].cpu().numpy() - ex['lam']).max():.3g}")
    assert np.abs(out["lam"].cpu().numpy() - ex["lam"]).max() < 2e-5
    assert np.abs(logp - ex["logp"]).max() < 5e-5
    # backward from the oracle's CTC gradient on the oracle's export, at this chunk
    lp_ref = torch.tensor(ex["logp"], requires_grad=True)
    _stock_ctc(torch, lp_ref, u["y_rel"], wl.input_lengths, wl.target_lengths, "cpu").backward()
    dl = lp_ref.grad.numpy()
    r = prunedctc.grouped_backward(H, W, uid, out["logp"], out["lam"], torch.from_numpy(dl.astype(np.float32)).cuda(),
                                   bias=bt, chunk=chunk, want_db=with_bias)
    fp32 = dtype == "f32"
    for name in ("dH", "dW") + (("db",) if with_bias else ()):
        got = r[name].cpu().numpy()
        e, c = rel_err(got, full[name]), cosine(got, full[name])
        say(f"  {name} rel={e:.3g} cos={c:.7f}")
        assert (e <= 1e-4) if fp32 else (c >= 0.99999)
    # the stock CTC on the GPU through the autograd wrapper
    Hg = H.clone().requires_grad_(True)
    Wg = W.clone().requires_grad_(True)
    bg = None if bt is None else bt.clone().requires_grad_(True)
    lp = prunedctc.grouped_head(Hg, Wg, uid, bg)
    loss = _stock_ctc(torch, lp, u["y_rel"], wl.input_lengths, wl.target_lengths, "cuda")
    loss.backward()
    lr = loss_rel(float(loss.item()), full["loss"])
    say(f"  stock CTC loss gpu={float(loss.item()):.9g} oracle={full['loss']:.9g} rel={lr:.3g}")
    assert lr <= (1e-5 if fp32 else 2e-3)
    for name, t in (("dH", Hg), ("dW", Wg)) + ((("db", bg),) if with_bias else ()):
        got = t.grad.float().cpu().numpy()
        c = cosine(got, full[name])
        say(f"  autograd {name} cos={c:.7f}")
        assert c >= (0.99999 if fp32 else 0.999)


def test_grouped_edges():
    """The selected ids cover the vocabulary (no merged class: its column is -inf); ids out
    of range or repeated are rejected."""
    import torch
    from paper_2609_33645_amd import prunedctc
    rng = np.random.default_rng(5)
    V, D, M = 24, 16, 70
    H = rng.standard_normal((M, D)).astype(np.float32)
    W = (rng.standard_normal((V, D)) * 0.4).astype(np.float32)
    perm = rng.permutation(V).astype(np.int32)
    ex = oracle.grouped_logprobs(H, W, perm)
    out = prunedctc.grouped_logprobs(torch.from_numpy(H).cuda(), torch.from_numpy(W).cuda(),
                                     torch.from_numpy(perm).cuda())
    logp = out["logp"].cpu().numpy()
    assert np.isneginf(logp[:, V]).all()
    assert np.abs(logp[:, :V] - ex["logp"]).max() < 5e-5
    dl = rng.standard_normal((M, V + 1)).astype(np.float32)
    dl[:, V] = 0.0
    dl[::3, :V] -= dl[::3, :V].mean(axis=1, keepdims=True)   # rows whose sum (g) is ~0
    dl[1::3, :V] = 0.0                                        # rows with no gradient at all
    r = prunedctc.grouped_backward(torch.from_numpy(H).cuda(), torch.from_numpy(W).cuda(), torch.from_numpy(perm).cuda(),
                                   out["logp"], out["lam"], torch.from_numpy(dl).cuda())
    ref = oracle.grouped_backward(H, W, ex["lam"], ex["logp"], dl[:, :V].astype(np.float64), perm)
    assert rel_err(r["dH"].cpu().numpy(), ref["dH"]) <= 1e-4
    assert rel_err(r["dW"].cpu().numpy(), ref["dW"]) <= 1e-4
    for bad in ([0, 3, 3], [0, V], [-1, 2]):
        with pytest.raises(prunedctc.PrunedCTCError) as e:
            prunedctc.grouped_logprobs(torch.from_numpy(H).cuda(), torch.from_numpy(W).cuda(),
                                       torch.tensor(bad, dtype=torch.int32, device="cuda"))
        assert e.value.code == -2


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_e2e_forecast_miss(dtype):
    """A -inf bias on one target label makes its utterance's loss infinite (status 2) although
    every normaliser is finite: the bf16 schedule's forecast of g is wrong for that utterance
    and the backward must still match the oracle (which excludes it)."""
    import torch
    from paper_2609_33645_amd import prunedctc
    wl = workloads.random_small(70, N=4, T_range=(30, 120), D=64, V=500, dtype=dtype, p_repeat=0.1, w_std=0.5)
    b = np.zeros(wl.V, np.float32)
    lab = int(wl.targets[wl.target_lengths[0] + 1])   # a label of utterance 1
    b[lab] = -np.inf
    say(f"forecast miss {dtype} label={lab} M={wl.M}")
    ref = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, wl.blank,
                         bias=b.astype(np.float64))
    assert ref["status"][1] == 2
    H, W, y = to_dev(wl)
    out = prunedctc.pruned_ctc_fwd_bwd(H, W, y, wl.input_lengths, wl.target_lengths, wl.blank, math.inf,
                                       bias=torch.from_numpy(b).cuda(), want_db=True)
    np.testing.assert_array_equal(out["status"].cpu().numpy(), ref["status"])
    assert loss_rel(float(out["loss"].item()), ref["loss"]) <= 1e-5
    for name in ("dH", "dW", "db"):
        got = out[name].cpu().numpy()
        assert np.isfinite(got).all(), name
        if dtype == "f32":
            assert rel_err(got, ref[name]) <= 1e-4, name
        else:
            assert cosine(got, ref[name]) >= 0.99999, name


def test_concurrent_calls_with_kernel_timing():
    """Kernel timing enabled while two host threads call the fused function at once: each timing
    scope owns its events until it closes, so the flush at the end of one thread's call never
    touches the other thread's open scopes.  Results equal those of the calls made alone, and
    every launch is counted exactly once (one normaliser launch per call)."""
    import threading
    import torch
    from paper_2609_33645_amd import prunedctc
    say("concurrent calls with kernel timing")
    wls = [workloads.random_small(95 + i, N=5, T_range=(40, 160), D=128, V=3000, dtype="bf16", p_repeat=0.1,
                                  beam=16.0, w_std=0.5) for i in range(2)]

    def call(wl):
        H, W, y = to_dev(wl)
        out = prunedctc.pruned_ctc_fwd_bwd(H, W, y, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam)
        torch.cuda.current_stream().synchronize()
        return [out["loss"].cpu(), out["dH"].cpu(), out["dW"].cpu()]

    alone = [call(wl) for wl in wls]
    calls = 4
    results = [[None] * calls for _ in wls]
    errors = []

    def worker(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for r in range(calls):
                    results[i][r] = call(wls[i])
        except Exception as e:  # reported below
            errors.append(repr(e))

    prunedctc.prof_reset()
    prunedctc.prof_enable(True)
    try:
        threads = [threading.Thread(target=worker, args=(i,)) for i in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join(timeout=100)
    finally:
        prunedctc.prof_enable(False)
    assert not any(t.is_alive() for t in threads)
    assert not errors, errors
    prof = prunedctc.prof_read()
    prunedctc.prof_reset()
    for i in range(2):
        for r in range(calls):
            for a, b in zip(results[i][r], alone[i]):
                assert torch.equal(a, b), (i, r)
    assert prof["lse_partial"]["launches"] == 2 * calls, prof["lse_partial"]
    # recompute launches (or, where the normaliser wrote a chunk's rows, its guard launch)
    nrc = sum(prof[k]["launches"] for k in ("recompute_dz", "recompute_check") if k in prof)
    assert nrc > 0 and nrc % (2 * calls) == 0, prof
    assert all(v["total_ms"] > 0 for v in prof.values())


# ---------------------------------------------------------------------------------------
# determinism: every reduction runs in a fixed order, also across the two streams
# ---------------------------------------------------------------------------------------

@pytest.mark.parametrize("dtype,D,chunk", [("bf16", 128, 1024), ("bf16", 2048, 768), ("f32", 136, 512)])
def test_e2e_bitwise_repeatable(dtype, D, chunk):
    import torch
    from paper_2609_33645_amd import prunedctc
    wl = workloads.random_small(81, N=5, T_range=(30, 160), D=D, V=3000, dtype=dtype, p_repeat=0.1, beam=16.0,
                                w_std=0.5 * math.sqrt(128 / D))
    rng = np.random.default_rng(5)
    bias = torch.from_numpy(rng.standard_normal(wl.V).astype(np.float32)).cuda()
    wts = torch.from_numpy(rng.uniform(0.5, 1.5, size=wl.N).astype(np.float32)).cuda()
    H, W, y = to_dev(wl)
    say(f"repeatable {dtype} M={wl.M} D={D} chunk={chunk}")
    outs = [prunedctc.pruned_ctc_fwd_bwd(H, W, y, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam, chunk=chunk,
                                         bias=bias, utt_weight=wts, want_db=True) for _ in range(2)]
    for k in ("loss", "loss_per_utt", "status", "dH", "dW", "db"):
        a, b = outs[0][k].cpu().numpy(), outs[1][k].cpu().numpy()
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), k
