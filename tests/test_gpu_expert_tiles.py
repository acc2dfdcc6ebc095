"""GPU parity of the expert tiles at the edges of their token passes.

One expert takes every token (E = 1, top_k = 1), so a tile's passes hold 1 to
8 token rows and the last pass of a larger batch holds the remainder. Float32
operands (z, p, u) enter the matrix cores as bf16 hi + lo halves in rows 0..7
and 8..15 of one product.

Tolerance: a split value is off by at most 2^-18 of itself, so an output is
off by 2^-18 of the sum of its terms' magnitudes, which for n = I
random-signed terms is about sqrt(2 n / pi) times the result's scale (8 to 31
here, 10 taken at least), with the float32 sums far below: 4e-5 to 1.2e-4. A
lost or misplaced lo half is 2^-9 of it, a hundred times more.
"""

import math

import numpy as np
import pytest
import torch

import oracle.cardan_oracle as O
from paper_2609_21137_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21137_amd import cardan
    return cardan


def _parity(C, H, I, E, k, d, K, r, B, seed, up_only=False, hot=0):
    print(f"[tiles] H={H} I={I} E={E} k={k} d={d} K={K} r={r} B={B} up_only={up_only} hot={hot}", flush=True)
    L = synth.make_layer(H, I, E, d, K, r, seed=seed, up_only=up_only, hot_experts=range(hot), hot_bias=6.0)
    x = synth.make_input(H, B, seed=seed)
    act = "relu2_up" if up_only else "silu_glu"
    y_ref, idx_ref, a_ref, margin = O.moe_layer_factored(x, L, k, d, act=act)
    assert np.all(margin > 1e-9)
    shape = C.make_shape(H, I, E, k, d, K, r)
    ws = C.new_workspace(shape, B)
    fn = C.moe_layer_relu2 if up_only else C.moe_layer
    y, idx, wt = fn(shape, C.bf16_tensor(x), C.DeviceLayer.from_numpy(L), ws=ws)
    torch.cuda.synchronize()
    assert C.workspace_status(ws) == 0, "an in-kernel wait timed out"
    assert np.array_equal(idx.cpu().numpy(), idx_ref)
    if hot:
        assert np.bincount(idx_ref.ravel(), minlength=E)[:hot].min() > 8  # several passes each
    err = np.abs(y.cpu().numpy().astype(np.float64) - y_ref).max() / np.abs(y_ref).max()
    print(f"[tiles] error {err:.2e}", flush=True)
    assert err <= 2.0 ** -18 * max(10.0, math.sqrt(2 * I / math.pi)), err


@pytest.mark.parametrize("r", (0, 8, 264))
@pytest.mark.parametrize("B", (1, 7, 8, 9, 16, 17, 33, 64))
@pytest.mark.parametrize("d", (2, 4, 8))
def test_token_passes(C, d, B, r):
    _parity(C, 192, 96, 1, 1, d, 256, r, B, seed=700 + B)


@pytest.mark.parametrize("B", (3, 8, 9))
def test_token_passes_up_only(C, B):
    _parity(C, 192, 160, 1, 1, 8, 200, 72, B, seed=740 + B, up_only=True)


@pytest.mark.parametrize("K", (1, 17, 255, 256))
@pytest.mark.parametrize("B", (1, 2))
@pytest.mark.parametrize("d", (2, 4, 8))
def test_code_book_sizes(C, d, B, K):
    """The book in LDS: packed words at batch 1 and d = 4, else one line of
    repeated words each; the words past K are zero."""
    _parity(C, 128, 64, 4, 2, d, K, 16, B, seed=760 + K)


@pytest.mark.parametrize("d", (2, 8))
def test_code_book_shorter_lines(C, d):
    """Eight token rows of 2432 inputs and 256 ranks leave room for lines of 64
    bytes only (the host sweep of the planner checks that they do)."""
    _parity(C, 2432, 288, 100, 8, d, 256, 256, 16, seed=780)


def test_code_book_lines_at_batch_one(C):
    """Tiles of two column groups have no batch-1 kernel: theirs reads the book
    as lines (the host sweep of the planner checks that this layer has them)."""
    _parity(C, 3968, 32, 32, 32, 8, 256, 256, 1, seed=790)


@pytest.mark.parametrize("B,k", ((1, 1), (2, 8), (3, 8), (7, 7), (8, 8), (13, 5), (16, 4), (65 // 13, 13)))
def test_routing_tables_from_lanes(C, B, k):
    """Selections held in lanes: 1 to 64 of them, on both sides of the 16 that
    one wave counts alone, and the first count beyond (65)."""
    _parity(C, 128, 64, 40, k, 8, 256, 8, B, seed=800 + B)


@pytest.mark.parametrize("S", (3, 17, 40, 64))
def test_routing_tables_repeats_and_invalid(C, S):
    """A caller's routing with repeated experts and invalid indices."""
    H, I, E, d, K, r, k = 128, 64, 5, 8, 256, 8, 1
    rng = np.random.default_rng(S)
    L = synth.make_layer(H, I, E, d, K, r, seed=820)
    x = synth.make_input(H, S, seed=820)
    idx = rng.integers(-1, E + 1, size=(S, k)).astype(np.int32)
    idx[0] = 2
    w = rng.random((S, k)).astype(np.float32)
    y_ref = np.zeros((S, H))
    z = np.stack([O.shared_proj(x, L["U_gate"]), O.shared_proj(x, L["U_up"])])
    xf = O.bf16_to_f64(x)
    for t in range(S):
        if 0 <= idx[t, 0] < E:
            Wg, Wu, Wd = (m for m in O.expert_matrices(L, int(idx[t, 0]), d))
            g, u = xf[t] @ Wg, xf[t] @ Wu
            y_ref[t] = w[t, 0] * ((O.silu(g) * u) @ Wd)
    shape = C.make_shape(H, I, E, k, d, K, r)
    ws = C.new_workspace(shape, S)
    y = C.vq_lr_expert_ffn(shape, C.bf16_tensor(x), torch.from_numpy(idx).cuda(), torch.from_numpy(w).cuda(),
                           torch.from_numpy(z.astype(np.float32)).cuda(), C.DeviceLayer.from_numpy(L), ws=ws)
    torch.cuda.synchronize()
    assert C.workspace_status(ws) == 0
    err = np.abs(y.cpu().numpy() - y_ref).max() / np.abs(y_ref).max()
    assert err <= 4e-5, err


@pytest.mark.parametrize("separate", (False, True))
@pytest.mark.parametrize("r", (8, 72, 512))
@pytest.mark.parametrize("B", (16, 17, 33, 64))
def test_shared_projection_token_groups(C, B, r, separate):
    """z = U^T x in groups of 16 tokens, one and several, whole and partial."""
    H = 320
    L = synth.make_layer(H, 32, 2, 8, 16, r, seed=840, separate_up_basis=separate)
    x = synth.make_input(H, B, seed=841)
    shape = C.make_shape(H, 32, 2, 1, 8, 16, r)
    ws = C.new_workspace(shape, B)
    Ug, Uu = C.bf16_tensor(L["U_gate"]), C.bf16_tensor(L["U_up"])
    for _ in range(2):  # the second call finds the flags as the first left them
        z = C.shared_proj(shape, C.bf16_tensor(x), Ug, Uu if separate else None, ws=ws)
    torch.cuda.synchronize()
    assert C.workspace_status(ws) == 0
    for got, U in zip(z.cpu().numpy(), (L["U_gate"], L["U_up"])):
        ref = O.shared_proj(x, U)
        # 320 float32 sums of exact products
        assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()


def test_noalloc_smaller_layout(C):
    """A layer whose usual layout exceeds the library's scratch array, but not
    the one with splits by bytes: it runs there with the latter and gives the
    usual result up to the order of the float32 sums."""
    H, I, E, k, d, K, r, B = 832, 1600, 8, 6, 4, 128, 112, 44
    L = C.DeviceLayer.from_numpy(synth.make_layer(H, I, E, d, K, r, seed=860))
    x = C.bf16_tensor(synth.make_input(H, B, seed=860))
    shape = C.make_shape(H, I, E, k, d, K, r)
    assert C.workspace_bytes(shape, B) > 16 << 20
    y, idx, _ = C.moe_layer(shape, x, L)
    y2, idx2, _ = C.moe_layer_noalloc(shape, x, L)
    torch.cuda.synchronize()
    assert torch.equal(idx, idx2)
    assert float((y - y2).abs().max()) <= 2e-5 * float(y.abs().max())


@pytest.mark.parametrize("B,k,E", ((9, 1, 2), (16, 2, 3), (17, 3, 4), (40, 5, 6), (64, 4, 5)))
@pytest.mark.parametrize("form", ("layer", "relu2", "dense"))
def test_experts_of_several_passes(C, form, B, k, E):
    """Experts of 8 to 64 tokens: a record, and so tiles of their own, for every
    8 of them, from both table builders (up to and over 64 selections)."""
    if form != "dense":
        _parity(C, 192, 96, E, k, 8, 256, 40, B, seed=880 + B, up_only=form == "relu2")
        return
    H, I = 192, 96
    L = synth.make_layer(H, I, E, 8, 1, 0, seed=890)
    W = synth.make_dense_weights(H, I, E, seed=890)
    x = synth.make_input(H, B, seed=890)
    y_ref, idx_ref, _, _ = O.moe_layer_dense(x, L["router_w"], L["router_bias"], W["W_gate"], W["W_up"],
                                             W["W_down"], k)
    dl = C.DenseLayer({"router_w": C.bf16_tensor(L["router_w"]), "router_bias": torch.from_numpy(L["router_bias"]).cuda(),
                       **{n: C.bf16_tensor(W[n]) for n in ("W_gate", "W_up", "W_down")}})
    y, idx, _ = C.dense_moe_layer(C.make_shape(H, I, E, k, 8, 1, 0), C.bf16_tensor(x), dl)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), idx_ref)
    assert np.abs(y.cpu().numpy() - y_ref).max() <= 4e-5 * np.abs(y_ref).max()


@pytest.mark.parametrize("H,I,up_only", ((576, 1024, False), (512, 1024, False), (576, 1280, True), (512, 1280, True)))
def test_wide_tiles_of_several_passes(C, H, I, up_only):
    """Down tiles of two column groups (odd and even counts of groups; the host
    sweep of the planner checks that these layers have them) of four experts
    that nearly every token selects: up to eight records each."""
    _parity(C, H, I, 96, 8, 8, 256, 136 if up_only else 24, 64, seed=900, up_only=up_only, hot=4)


@pytest.mark.parametrize("d,B,E,k", ((8, 17, 3, 2), (4, 40, 6, 5)))
def test_dense_down_of_several_passes(C, d, B, E, k):
    H, I, r = 320, 160, 40
    L = synth.make_layer(H, I, E, d, 256, r, seed=910)
    Wd = synth.make_dense_weights(H, I, E, 910, which=("down",))["W_down"]
    x = synth.make_input(H, B, seed=910)
    y_ref, idx_ref, _, margin = O.moe_layer_dense_down(x, L, Wd, k, d)
    assert np.all(margin > 1e-9) and np.bincount(idx_ref.ravel()).max() > 8
    ws = C.new_workspace(C.make_shape(H, I, E, k, d, 256, r), B)
    y, idx, _ = C.moe_layer_dense_down(C.make_shape(H, I, E, k, d, 256, r), C.bf16_tensor(x), C.DeviceLayer.from_numpy(L),
                                       C.bf16_tensor(Wd), ws=ws)
    torch.cuda.synchronize()
    assert C.workspace_status(ws) == 0
    assert np.array_equal(idx.cpu().numpy(), idx_ref)
    assert np.abs(y.cpu().numpy() - y_ref).max() <= 2.0 ** -18 * max(10.0, math.sqrt(2 * I / math.pi)) * np.abs(y_ref).max()


# the last: passes of 4 token rows (the host sweep of the planner checks it)
@pytest.mark.parametrize("H,I,E,k,d,r,B", ((192, 96, 3, 2, 8, 40, 16), (192, 96, 5, 4, 4, 72, 33), (192, 96, 3, 2, 2, 8, 17),
                                          (4416, 32, 300, 2, 8, 80, 16)))
def test_step_of_several_passes(C, H, I, E, k, d, r, B):
    """A stack of two layers whose experts take up to 33 tokens: the split
    operands' parts as two products. The oracle of each layer takes the
    step's own input; the second layer's is checked in the step's tests."""
    Ls = [synth.make_layer(H, I, E, d, 256, r, seed=920, layer=l, hot_experts=range(2), hot_bias=6.0) for l in range(2)]
    x = synth.make_input(H, B, seed=920)
    shape = C.make_shape(H, I, E, k, d, 256, r)
    ws = C.new_workspace(shape, B)
    xn = torch.empty((1, B, H), dtype=torch.bfloat16, device="cuda")
    print(f"[tiles] step H={H} I={I} E={E} k={k} d={d} r={r} B={B}", flush=True)
    y, idx, _ = C.moe_decode_step(shape, C.bf16_tensor(x), [C.DeviceLayer.from_numpy(L) for L in Ls], 1e-6, ws=ws, x_norm=xn)
    torch.cuda.synchronize()
    assert C.workspace_status(ws) == 0
    y0, idx0, _, m0 = O.moe_layer_factored(x, Ls[0], k, d)
    y1, idx1, _, m1 = O.moe_layer_factored(C.bf16_bits(xn[0]), Ls[1], k, d)
    assert min(m0.min(), m1.min()) > 1e-9
    for got, ref in zip(idx.cpu().numpy(), (idx0, idx1)):
        assert np.array_equal(got, ref) and np.bincount(ref.ravel()).max() > 8
    tol = 2.0 ** -18 * max(10.0, math.sqrt(2 * I / math.pi))
    assert np.abs(y.cpu().numpy() - y1).max() <= tol * np.abs(y1).max()
    xr = O.rmsnorm(y0, 1e-6)
    # one bf16 step, and y0's own error through the normalisation
    assert np.all(np.abs(O.bf16_to_f64(C.bf16_bits(xn[0])) - xr) <= 2.0 ** -8 * np.abs(xr) + 2 * tol * np.abs(xr).max())


@pytest.mark.parametrize("bad", (float("inf"), float("nan")))
@pytest.mark.parametrize("d,r", ((8, 40), (4, 0)))
def test_non_finite_tokens_stay_apart(C, d, r, bad):
    """A value that is not finite reaches every output of its token (its hi and
    lo parts are rows of one product) and no bit of another token's."""
    H, I, B = 192, 96, 19
    shape = C.make_shape(H, I, 1, 1, d, 256, r)
    DL = C.DeviceLayer.from_numpy(synth.make_layer(H, I, 1, d, 256, r, seed=930))
    x = C.bf16_tensor(synth.make_input(H, B, seed=930))
    idx, w = torch.zeros((B, 1), dtype=torch.int32, device="cuda"), torch.ones((B, 1), device="cuda")
    z = C.shared_proj(shape, x, DL.tensors["U_gate"], DL.tensors["U_up"]) if r else None
    ws = C.new_workspace(shape, B)
    ref = C.vq_lr_expert_ffn(shape, x, idx, w, z, DL, ws=ws)
    hit = [0, 5, 7, 8, 18]
    x2, z2 = x.clone(), z.clone() if r else None
    for t in hit:
        if r and t != 5:
            z2[:, t, t] = bad
        else:
            x2[t, 3 * t] = bad
    y = C.vq_lr_expert_ffn(shape, x2, idx, w, z2, DL, ws=ws)
    torch.cuda.synchronize()
    assert C.workspace_status(ws) == 0
    rest = [t for t in range(B) if t not in hit]
    assert torch.isfinite(ref).all() and torch.equal(y[rest], ref[rest])
    assert not torch.isfinite(y[hit]).any()


@pytest.mark.parametrize("H,I,E,k,d,r,B", ((64, 672, 64, 32, 4, 424, 64), (64, 1152, 64, 16, 2, 512, 64),
                                          (1536, 416, 64, 29, 8, 504, 64)))
def test_layers_near_the_lds_limit(C, H, I, E, k, d, r, B):
    """Large routing tables beside long tiles of many ranks: 80 to 96 KB of LDS."""
    _parity(C, H, I, E, k, d, 256, r, B, seed=940)
