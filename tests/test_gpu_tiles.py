"""GPU kernels at the sizes where their tiling can go wrong, against the fp64 oracle: edges of
tiles and of slices, remainders, the smallest and the largest of a rule's range."""
from __future__ import annotations

import math

import numpy as np
import pytest

import oracle
from paper_2609_33645_amd import workloads
from tests.gpu_util import cosine, loss_rel, rel_err, run_gpu, say, to_dev

pytestmark = pytest.mark.gpu


def _fixed(dtype, T, D, V, seed, blank=0, u_frac=0.2, w_std=None):
    T = np.asarray(T, np.int32)
    return workloads.synthesize(name="tiles", dtype=dtype, T=T, U=(T * u_frac).astype(np.int32), D=D, V=V,
                                rng=np.random.default_rng(seed), token_law="uniform", blank=blank, w_std=w_std)


# ---- fp32 products on the split engine ----------------------------------------------------------

@pytest.mark.parametrize("T,D,V,chunk", [
    ([1], 8, 2, 0),                  # one frame, half a k-tile, one ragged tile of two classes
    ([255], 16, 255, 0),             # one k-tile; a frame and a class short of whole tiles
    ([256], 24, 256, 0),             # whole tiles, one k-tile and a half
    ([200, 57], 264, 257, 256),      # one past whole tiles in frames, width and classes; two chunks
    ([40] * 30, 520, 1025, 512),     # a narrower last chunk (one class) on the first chunk's dH slices
    ([100] * 30, 64, 700, 256),      # the frames of dW in slices
])
def test_f32_tile_edges(T, D, V, chunk):
    wl = _fixed("f32", T, D, V, 5 + D + V, blank=V - 1)
    say(f"f32 tile edges M={wl.M} D={D} V={V} chunk={chunk}")
    ref = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam)
    res = run_gpu(wl, chunk=chunk)
    np.testing.assert_array_equal(res["status"], ref["status"])
    assert loss_rel(res["loss"], ref["loss"]) <= 1e-5
    # every product is rounded to about 2^-24 and summed in fp32: far inside the stated 1e-4
    assert rel_err(res["dH"], ref["dH"]) <= 1e-5
    assert rel_err(res["dW"], ref["dW"]) <= 1e-5


@pytest.mark.parametrize("e", [100, -90])
def test_f32_split_keeps_the_range(e):
    """H 2^e and W 2^-e give the very same logits as H and W (powers of two move through the splits
    and the sums exactly while every part stays a normal number), and values at the top of fp32's
    range give finite logits: split (3.3e38) and, where they round to infinity in bf16 (3.4e38), on
    the fp32 instructions."""
    import torch

    from paper_2609_33645_amd import prunedctc
    wl = _fixed("f32", [70], 72, 300, 3)
    H, W, _ = to_dev(wl)
    a = prunedctc.lse_select(H, W)["lam"]
    b = prunedctc.lse_select(H * 2.0 ** e, W * 2.0 ** -e)["lam"]
    assert torch.equal(a, b)
    W[:, 0] = 1e-38
    # 1e-38 splits into parts down to 2^-142, below bf16's smallest: its product is good to 2^-8; on
    # the fp32 instructions it is rounded like any other
    for top, bar in ((3.3e38, 3.4 * 2.0 ** -8), (3.4e38, 1e-5)):
        H[:, 0] = top
        c = prunedctc.lse_select(H, W)["lam"].cpu().numpy()
        ref = oracle.log_normalizer(H.cpu().numpy().astype(np.float64), W.cpu().numpy().astype(np.float64))
        assert np.abs(c - ref).max() <= bar


@pytest.mark.parametrize("chunk", [0, 256])
def test_f32_gradients_of_the_least_probabilities(chunk):
    """Classes whose probabilities come near fp32's least (7e-34 to 7e-38) have gradient rows and bias
    gradients with an error of the exponent's rounding: 2^-18 at 124 binary places."""
    import torch

    from paper_2609_33645_amd import prunedctc
    wl = _fixed("f32", [90, 41], 40, 700, 8, u_frac=0.1, w_std=0.02)
    b = np.zeros(700, np.float32)
    rare = np.setdiff1d(np.arange(1, 700, 9), wl.targets)
    b[rare] = -np.linspace(70, 79, rare.size)  # the logits themselves are within 1 of each other
    H, W, y = to_dev(wl)
    out = prunedctc.pruned_ctc_fwd_bwd(H, W, y, wl.input_lengths, wl.target_lengths, 0, wl.beam, chunk=chunk,
                                       bias=torch.from_numpy(b).cuda(), want_db=True)
    ref = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, 0, wl.beam, bias=b)
    dW, db = out["dW"].cpu().numpy()[rare], out["db"].cpu().numpy()[rare]
    scale = np.abs(ref["dW"][rare]).max(1, keepdims=True)
    say(f"least probabilities: largest dW row {scale.max():.2g}, least {scale.min():.2g}")
    assert scale.min() < 5e-36
    assert (np.abs(dW - ref["dW"][rare]) / scale).max() <= 3 * 2.0 ** -18
    assert np.abs(db / ref["db"][rare] - 1).max() <= 3 * 2.0 ** -18


def test_f32_split_drops_less_than_a_rounding():
    """Logits that are one product, of values chosen so that a first part cut to bf16 instead of
    rounded would drop the most (2^-22.4 of the product): the mean error, in which roundings cancel,
    shows what is dropped (below 2^-24.2 for any product with parts rounded to nearest)."""
    import torch

    from paper_2609_33645_amd import prunedctc

    def rest(x, nearest):
        """x minus its first part, that minus its own, of float32 values as float64."""
        out = []
        for near in (nearest, True):
            u = x.astype(np.float32).view(np.uint32).astype(np.uint64)
            u = u + 0x7fff + ((u >> 16) & 1) if near else u
            x = x - (u & 0xffff0000).astype(np.uint32).view(np.float32)
            out.append(x)
        return out

    def dropped(a, b, nearest):
        (a1, a2), (b1, b2) = rest(a, nearest), rest(b, nearest)
        return ((a1 - a2) * b2 + a2 * (b1 - b2) + a2 * b2) / (a * b)

    rng = np.random.default_rng(3)
    a, b = ((1.0 + rng.random(300_000) * 0.0625).astype(np.float32).astype(np.float64) for _ in range(2))
    err = []
    for x in b[np.argsort(-dropped(a, b, False))[:20]]:
        top = a[np.argsort(-dropped(a, np.full_like(a, x), False))[:1000]]
        assert dropped(top, x * np.ones(1000), False).min() > 2.0 ** -23
        assert np.abs(dropped(top, x * np.ones(1000), True)).max() < 2.0 ** -24.2
        H, W = torch.zeros(1000, 8), torch.zeros(2, 8)
        H[:, 0] = torch.from_numpy(top * 64).float()
        W[0, 0] = float(x)  # logits (a x, 0): lambda = a x + log(1 + exp(-a x)), within 2^-92 of a x
        lam = prunedctc.lse_select(H.cuda(), W.cuda())["lam"].cpu().numpy()
        err.append(lam / (top * 64 * x) - 1.0)
    say(f"mean error {np.mean(err):.3g}, largest {np.abs(err).max():.3g}")
    assert abs(np.mean(err)) <= 2.0 ** -24.2
    assert np.abs(err).max() <= 3 * 2.0 ** -24  # dropped, the sum's rounding, the exponent's in lambda


@pytest.mark.parametrize("V", [300, 513])
def test_f32_infinite_operands(V):
    """An infinite weight (a class masked or forced by its weights) acts as in fp32 arithmetic: a
    logit of -inf has probability 0, one of +inf wins the argmax, and everything else is as it is
    without it."""
    import torch

    from paper_2609_33645_amd import prunedctc
    wl = _fixed("f32", [70], 40, V, 21)
    wl.H[:, 3] = np.abs(wl.H[:, 3]) + 0.1
    masked = V - 2
    assert masked not in wl.targets
    wl.W[masked, 3] = -np.inf
    H, W, y = to_dev(wl)
    Z = wl.H.astype(np.float64) @ np.delete(wl.W, masked, 0).astype(np.float64).T
    lam = Z.max(1) + np.log(np.exp(Z - Z.max(1, keepdims=True)).sum(1))
    out = prunedctc.lse_select(H, W, torch.tensor([0, masked], dtype=torch.int32, device="cuda"))
    assert np.abs(out["lam"].cpu().numpy() - lam).max() <= 1e-5
    assert torch.isneginf(out["S"][:, 1]).all()
    assert np.abs(out["S"][:, 0].cpu().numpy() - (Z[:, 0] - lam)).max() <= 1e-5
    # the loss and the weights' gradients, as without the masked class (its own row is zero); dH is
    # compared where the infinite weight does not meet the class's zero probability
    res = run_gpu(wl)
    y2 = np.where(wl.targets > masked, wl.targets - 1, wl.targets)
    ref = oracle.fwd_bwd(wl.H, np.delete(wl.W, masked, 0), y2, wl.input_lengths, wl.target_lengths, 0, wl.beam)
    assert loss_rel(res["loss"], ref["loss"]) <= 1e-5
    assert rel_err(np.delete(res["dW"], masked, 0), ref["dW"]) <= 1e-5 and not res["dW"][masked].any()
    assert rel_err(np.delete(res["dH"], 3, 1), np.delete(ref["dH"], 3, 1)) <= 1e-5
    # +inf where the frame's value is positive, -inf where it is negative
    W[masked, 3] = 0.0
    W[1, 7] = np.inf
    ids = prunedctc.greedy_decode(H, W, [70])["ids"].cpu().numpy()
    Z = wl.H.astype(np.float64) @ W.cpu().numpy().astype(np.float64).T
    assert np.all(ids[wl.H[:, 7] > 0] == 1)
    rest = Z[wl.H[:, 7] < 0]
    np.testing.assert_array_equal(ids[wl.H[:, 7] < 0], rest.argmax(1))


def test_f32_largest_frame_values():
    """Values that round to infinity in bf16 in the weights' product too (frames of 3.4e38 where the
    weights are zero, a loss weight of 1e-20): on the fp32 instructions, and as the oracle has it."""
    import torch

    from paper_2609_33645_amd import prunedctc
    wl = _fixed("f32", [300, 41], 40, 300, 23, w_std=0.2)
    wl.W[:, 5] = 0.0
    wl.H[::3, 5] = 3.4e38
    w = np.full(2, 1e-20, np.float32)
    H, W, y = to_dev(wl)
    out = prunedctc.pruned_ctc_fwd_bwd(H, W, y, wl.input_lengths, wl.target_lengths, 0, wl.beam,
                                       utt_weight=torch.from_numpy(w).cuda())
    ref = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, 0, wl.beam, weights=w)
    assert loss_rel(float(out["loss"].item()), ref["loss"]) <= 1e-5
    dW, dH = out["dW"].cpu().numpy(), out["dH"].cpu().numpy()
    assert rel_err(dW[:, 5], ref["dW"][:, 5]) <= 1e-5 and np.abs(ref["dW"][:, 5]).max() > 1e17
    assert rel_err(np.delete(dW, 5, 1), np.delete(ref["dW"], 5, 1)) <= 1e-5
    assert rel_err(dH, ref["dH"]) <= 1e-5


# ---- discarded mass of several beams in one launch ----------------------------------------------

@pytest.mark.parametrize("nbeams", [1, 2, 9, 10, 20])
def test_discarded_mass_beam_groups(nbeams):
    """Nine beams share a launch: around that number, each beam's row against the oracle."""
    import torch

    from paper_2609_33645_amd import prunedctc
    rng = np.random.default_rng(nbeams)
    T, U = np.array([30, 1, 90, 17], np.int32), np.array([6, 0, 40, 16], np.int32)
    K = 23
    y = rng.integers(1, K, size=int(U.sum())).astype(np.int32)
    S = workloads.random_scores(nbeams, int(T.sum()), K, integer=True)  # margins are integers ..
    beams = [0.5 + 3 * b for b in range(nbeams)]                       # .. and thresholds between them
    got = prunedctc.discarded_mass(torch.from_numpy(S).cuda(), torch.from_numpy(y).cuda(), T, U, beams).cpu().numpy()
    ref = oracle.discarded_mass(S.astype(np.float64), y, T, U, beams)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    # each sum is of products of T float exponentials (2^-24 each), both recursions on the same ones
    assert np.nanmax(np.abs(got - ref)) <= 90 * 2.0 ** -23


# ---- few frames: shorter normaliser runs and more dH slices (bf16) ------------------------------

@pytest.mark.parametrize("T,D,V", [
    ([300], 128, 40_000),   # runs of a few tiles, up to 32 dH slices, the first chunk from the normaliser
    ([40], 256, 20_001),    # one frame tile; a ragged last partition
    ([130, 130], 520, 9000),  # not a multiple of 128: no E chunk, partial k-tiles
])
def test_few_frames_slices(T, D, V):
    wl = _fixed("bf16", T, D, V, 11 + D, u_frac=0.1, w_std=0.5 * math.sqrt(128 / D))
    say(f"few frames M={wl.M} D={D} V={V}")
    ref = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam)
    res = run_gpu(wl)
    assert loss_rel(res["loss"], ref["loss"]) <= 1e-5
    # only dZ is rounded to bf16 (2^-9 a value): the suite's tight bar
    assert cosine(res["dH"], ref["dH"]) >= 0.99999
    assert cosine(res["dW"], ref["dW"]) >= 0.99999


@pytest.mark.parametrize("D,V", [(256, 20_001), (256, 60_001), (72, 20_001), (2048, 700)])
def test_lse_select_does_not_depend_on_the_batch(D, V):
    """A frame's lambda and S are the same, to the last bit, alone and in a batch: S decides the
    arcs at a beam's edge, where its last bit moves the discarded mass."""
    import torch

    from paper_2609_33645_amd import prunedctc
    wl = _fixed("bf16", [8200], D, V, 17, u_frac=0.0)
    H, W, _ = to_dev(wl)
    u = torch.arange(0, V, 37, dtype=torch.int32, device="cuda")
    all_ = prunedctc.lse_select(H, W, u)
    for m in (1, 40, 300, 1500):
        few = prunedctc.lse_select(H[:m], W, u)
        assert torch.equal(few["lam"], all_["lam"][:m]) and torch.equal(few["S"], all_["S"][:m]), m


@pytest.mark.parametrize("M,V", [(1, 700), (150, 50_000), (257, 2500), (6700, 8931), (8192, 9000), (4000, 2300)])
def test_greedy_few_frames(M, V):
    from paper_2609_33645_amd import prunedctc
    wl = _fixed("bf16", [M], 128, V, M, u_frac=0.0)
    H, W, _ = to_dev(wl)
    ids = prunedctc.greedy_decode(H, W, [M])["ids"].cpu().numpy()
    Z = wl.H.astype(np.float64) @ wl.W.astype(np.float64).T
    top = Z.max(1)
    # the products' rounding (fp32 sums of 128 products) may pick another class within it
    assert np.all(Z[np.arange(M), ids] >= top - 1e-5 * np.abs(top))


# ---- lattice passes over one and four wavefronts --------------------------------------------------

@pytest.mark.parametrize("U", [0, 31, 63, 64, 127, 128, 255, 256, 384, 512, 700, 767, 768, 1022])
@pytest.mark.parametrize("beam", [math.inf, 6.5])
def test_lattice_wavefront_edges(U, beam):
    """Targets around every change of the states per lane and of the wavefront count, with repeated
    labels at the wavefronts' edges, beside a short utterance: losses, occupancies and kept arcs."""
    import torch

    from paper_2609_33645_amd import prunedctc
    rng = np.random.default_rng(U)
    Us = np.array([U, 3], np.int32)
    K = 40
    y = rng.integers(1, K, size=int(Us.sum())).astype(np.int32)
    y[1:U][rng.random(max(U - 1, 0)) < 0.2] = 1
    T = np.array([U + int((y[1:U] == y[:U - 1][:max(U - 1, 0)]).sum()) + 23, 9], np.int32)
    S = workloads.random_scores(U + 1, int(T.sum()), K, integer=True)  # margins >= 0.499 from the beam
    say(f"lattice edges T={T.tolist()} U={U} beam={beam}")
    ref = oracle.ctc_from_scores(S.astype(np.float64), y, T, Us, beam=beam)
    out = prunedctc.ctc_dp(torch.from_numpy(S).cuda(), torch.from_numpy(y).cuda(), T, Us, beam=beam,
                           want_mask=math.isfinite(beam))
    np.testing.assert_array_equal(out["status"].cpu().numpy(), ref["status"])
    np.testing.assert_allclose(out["loss_per_utt"].cpu().numpy(), ref["loss_n"], rtol=2e-6)
    # the tables keep each state's score below its frame's best in float32 (2^-24 relative, in alpha
    # and in beta), and the state an alignment needs may lie that far below: at most the sum of the
    # utterance's scores, each frame's largest magnitude counted
    depth = float(np.abs(S[:T[0]]).max(1).sum())
    assert np.abs(out["G"].cpu().numpy() - ref["G"]).max() < 2e-5 + 2.0 ** -23 * depth
    if math.isfinite(beam):
        mask, base = out["mask"].cpu().numpy(), 0
        for n in range(2):
            if ref["status"][n] != 0:
                base += int(T[n]) * (2 * int(Us[n]) + 1)
                continue
            Sp, mg = 2 * int(Us[n]) + 1, ref["per_utt"][n]["margins"]
            stay = mg["stay"].copy()
            stay[0] = mg["start"]
            want = (stay >= 0) | ((mg["step"] >= 0) << 1) | ((mg["skip"] >= 0) << 2)
            want[T[n] - 1] |= (mg["final"] >= 0) << 3
            np.testing.assert_array_equal(mask[base:base + int(T[n]) * Sp].reshape(int(T[n]), Sp), want)
            base += int(T[n]) * Sp


@pytest.mark.parametrize("beam", [math.inf, 6.5])
def test_lattice_wavefronts_with_excluded_utterances(beam):
    """Four-wavefront lattices whose total is not finite (status 2, set by the forward pass while
    backward passes of the same launch are still to begin: more workgroups than fit at once) among
    others: statuses, zero rows, and the others as they are alone."""
    import torch

    from paper_2609_33645_amd import prunedctc
    N, U, K = 400, 130, 40
    rng = np.random.default_rng(9)
    y = rng.integers(1, K, size=N * U).astype(np.int32)
    T = np.full(N, 3 * U, np.int32)
    S = workloads.random_scores(9, int(T.sum()), K, integer=True).reshape(N, 3 * U, K)
    bad = np.arange(N) % 3 != 0
    S[bad, -1] = -np.inf  # no alignment has a finite score ..
    S[bad & (np.arange(N) % 2 == 0), -2, 0] = np.nan  # .. or is a number
    dev = lambda n: (torch.from_numpy(S[n].reshape(-1, K)).cuda(),  # noqa: E731
                     torch.from_numpy(y.reshape(N, U)[n].reshape(-1)).cuda())
    say(f"excluded utterances beam={beam}")
    out = prunedctc.ctc_dp(*dev(np.arange(N)), T, np.full(N, U), beam=beam)
    np.testing.assert_array_equal(out["status"].cpu().numpy(), np.where(bad, 2, 0))
    G = out["G"].cpu().numpy().reshape(N, 3 * U, K)
    assert not G[bad].any()
    for n in (0, 3, 198, 399):
        alone = prunedctc.ctc_dp(*dev(np.array([n])), T[:1], [U], beam=beam)
        np.testing.assert_array_equal(G[n], alone["G"].cpu().numpy())
        assert float(alone["loss_per_utt"][0]) == float(out["loss_per_utt"][n])


@pytest.mark.parametrize("U", [63, 64, 127, 128, 300, 520, 800])
def test_discarded_mass_wavefront_edges(U):
    import torch

    from paper_2609_33645_amd import prunedctc
    rng = np.random.default_rng(U)
    K, Us = 30, np.array([U], np.int32)
    y = rng.integers(1, K, size=U).astype(np.int32)
    # three frames a label: the recursion's doubles, scaled by the frame's largest, keep the final
    # states while they lie within 2^1000 of it (targets that nearly fill their frames may not)
    T = np.array([3 * U + 15], np.int32)
    S = workloads.random_scores(U, int(T[0]), K, integer=True)
    beams = [2.5, 7.5]
    got = prunedctc.discarded_mass(torch.from_numpy(S).cuda(), torch.from_numpy(y).cuda(), T, Us, beams).cpu().numpy()
    ref = oracle.discarded_mass(S.astype(np.float64), y, T, Us, beams)
    # T float emission factors (2^-23 each, the same in both recursions)
    assert np.abs(got - ref).max() <= float(T[0]) * 2.0 ** -23


# ---- union in one launch (small vocabularies) and in two ------------------------------------------

@pytest.mark.parametrize("V", [2, 2047, 2048, 2049, 4096, 32_767, 32_768, 32_769])
def test_union_block_edges(V):
    import torch

    from paper_2609_33645_amd import prunedctc
    rng = np.random.default_rng(V)
    blank = int(rng.integers(0, V))
    ids = rng.integers(0, V - 1, size=500)
    ids = np.where(ids >= blank, ids + 1, ids)
    ids[:3] = [v for v in (0, V - 1, (V - 1) // 2048 * 2048) if v != blank][0]  # a block's first or last class
    y = torch.from_numpy(ids.astype(np.int32)).cuda()
    out = prunedctc.union_remap(y, blank, V)
    ref = oracle.union_remap(ids, np.array([ids.size]), blank=blank, V=V)
    np.testing.assert_array_equal(out["u_ids"].cpu().numpy(), ref["u_ids"])
    np.testing.assert_array_equal(out["remap"].cpu().numpy(), ref["remap"])
    np.testing.assert_array_equal(out["y_rel"].cpu().numpy(), ref["y_rel"])
    bad = y.clone()
    bad[7] = V
    with pytest.raises(prunedctc.PrunedCTCError) as err:
        prunedctc.union_remap(bad, blank, V)
    assert err.value.code == -2


# ---- frames from H transposed: argmax and normaliser with bias -------------------------------------

@pytest.mark.parametrize("M,V,bias", [(513, 2000, False), (700, 2305, True), (512, 300, True),
                                      (5210, 59_990, False), (5201, 60_100, True)])  # the last two transposed
def test_greedy_transposed_frames(M, V, bias):
    import torch

    from paper_2609_33645_amd import prunedctc
    wl = _fixed("bf16", [M], 256, V, M + V, u_frac=0.0)
    H, W, _ = to_dev(wl)
    b = np.random.default_rng(1).standard_normal(V).astype(np.float32) if bias else np.zeros(V, np.float32)
    ids = prunedctc.greedy_decode(H, W, [M], bias=torch.from_numpy(b).cuda() if bias else None)["ids"].cpu().numpy()
    Z = wl.H.astype(np.float64) @ wl.W.astype(np.float64).T + b
    top = Z.max(1)
    # the products' rounding (fp32 sums of 256 products) may pick another class within it
    assert np.all(Z[np.arange(M), ids] >= top - 1e-5 * np.abs(top))


@pytest.mark.parametrize("D", [256, 1024])
def test_greedy_workspace_sizes(D):
    """The same ids and tokens with the smallest workspace (D = 256: H transposed in what the
    partials leave; D = 1024: none) and with room for H transposed (from M V D = 8e10 on)."""
    import ctypes

    import torch

    from paper_2609_33645_amd import prunedctc
    L, N = prunedctc.lib(), 2
    V = int(8e10 / D / 3701) + 1
    wl = _fixed("bf16", [400, 3301], D, V, D, u_frac=0.0, w_std=0.1)
    H, W, _ = to_dev(wl)
    T, M = wl.input_lengths, wl.M
    least, most = L.pctc_greedy_workspace_size(N, M, D), L.pctc_greedy_workspace_size_ex(1, N, M, D, V)
    assert (most > least) == (D == 1024)
    assert L.pctc_greedy_workspace_size_ex(1, N, M, D, V - 1) == least
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    got = []
    for size in (least, most):
        ws = prunedctc._workspace(size, H.device)
        ids, tok, n = (torch.full((k,), -7, dtype=torch.int32, device="cuda") for k in (M, M, N))
        assert L.pctc_greedy_decode(1, p(H), D, p(W), None, V, prunedctc._i32p(T), N, 0, p(ids), p(tok), p(n), p(ws),
                                    ctypes.c_size_t(size), prunedctc._stream(None)) == 0
        got.append((ids, tok, n))
    assert all(torch.equal(a, b) for a, b in zip(*got))
    ws = prunedctc._workspace(least, H.device)
    assert L.pctc_greedy_decode(1, p(H), D, p(W), None, V, prunedctc._i32p(T), N, 0, None, p(tok), p(n), p(ws),
                                ctypes.c_size_t(least - 1), prunedctc._stream(None)) == -4


@pytest.mark.parametrize("T,V", [([256] * 8, 2000), ([250] * 9, 2305)])
def test_fused_bias_transposed_frames(T, V):
    """The biased normaliser of the fused call on both sides of its rule (2,048 and 2,250 frames)."""
    wl = _fixed("bf16", T, 512, V, V, u_frac=0.1, w_std=0.05)
    b = np.random.default_rng(6).standard_normal(V).astype(np.float32)
    say(f"fused bias M={wl.M} V={V}")
    ref = oracle.fwd_bwd(wl.H, wl.W, wl.targets, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam, bias=b)
    import torch

    from paper_2609_33645_amd import prunedctc
    H, W, y = to_dev(wl)
    out = prunedctc.pruned_ctc_fwd_bwd(H, W, y, wl.input_lengths, wl.target_lengths, wl.blank, wl.beam,
                                       bias=torch.from_numpy(b).cuda(), want_db=True)
    assert loss_rel(float(out["loss"].item()), ref["loss"]) <= 1e-5
    for k in ("dH", "dW", "db"):
        assert cosine(out[k].cpu().numpy(), ref[k]) >= 0.99999, k


@pytest.mark.parametrize("M,D,V", [(70, 128, 700), (300, 256, 2049), (33, 72, 300), (260, 2048, 513),
                                   (2048, 512, 700), (2049, 512, 2305), (2100, 640, 300)])
def test_grouped_bias_normaliser(M, D, V):
    """The complement's normaliser with its -inf bias (frames from H transposed for more than 2,048
    frames where D is a multiple of 128, from 512 on, and below the wide heads)."""
    import torch

    from paper_2609_33645_amd import prunedctc
    wl = _fixed("bf16", [M], D, V, M + D, u_frac=0.0)
    H, W, _ = to_dev(wl)
    g = np.random.default_rng(D)
    u = np.concatenate([[0], 1 + np.sort(g.choice(V - 1, 20, replace=False))]).astype(np.int32)
    b = torch.from_numpy(g.standard_normal(V).astype(np.float32)).cuda()
    ud = torch.from_numpy(u).cuda()
    f = prunedctc.grouped_logprobs(H, W, ud, b)
    ref = oracle.grouped_logprobs(wl.H, wl.W, u, bias=b.cpu().numpy())
    assert np.abs(f["lam"].cpu().numpy() - ref["lam"]).max() < 2e-5
    assert np.abs(f["logp"].cpu().numpy() - ref["logp"]).max() < 5e-5


def test_grouped_fp32_many_classes():
    """An fp32 export of more classes than 32 tiles a partition: partitions of any length."""
    import torch

    from paper_2609_33645_amd import prunedctc
    M, D, V = 3, 8, 2_200_000
    g = np.random.default_rng(4)
    H = g.standard_normal((M, D)).astype(np.float32)
    W = (g.standard_normal((V, D)) * 0.3).astype(np.float32)
    b = g.standard_normal(V).astype(np.float32)
    u = np.array([7, 1, 1_100_000, V - 1], np.int32)
    say(f"grouped fp32 V={V}")
    f = prunedctc.grouped_logprobs(*(torch.from_numpy(x).cuda() for x in (H, W, u, b)))
    ref = oracle.grouped_logprobs(H, W, u, bias=b)
    assert np.abs(f["lam"].cpu().numpy() - ref["lam"]).max() < 2e-5
    assert np.abs(f["logp"].cpu().numpy() - ref["logp"]).max() < 5e-5
