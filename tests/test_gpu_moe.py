"""Parity of the dispatch, expert-network, combine and MoE-forward kernels with the
oracle (Mixture-of-Experts, Eq. 1, with SwiGLU or two-layer ReLU expert networks), on
seeded routing."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2508_06024_amd import ec2moe as E
from paper_2508_06024_amd import workload as W
from tests.gpu_common import assert_close, down, say, tol, up, up_f32, up_i32

pytestmark = pytest.mark.gpu


# ----------------------------------------------------------------------------- permutation

PERM_CASES = [
    # T, M, k, n_keep, skew
    (64, 8, 2, 6, 0.0),
    (1024, 16, 2, 12, 0.0),
    (8192, 64, 6, 48, 1.1),     # 49152 assignments, chunked kernels, Zipf-skewed
    (4097, 8, 2, 8, 0.0),       # ragged last chunk
    (1, 4, 1, 4, 0.0),
    (3000, 256, 16, 256, 0.5),  # maximum experts and top-k
    (32, 64, 8, 16, 0.0),
    (8192, 8, 1, 8, 0.0),       # largest single-workgroup input
    (4097, 16, 2, 12, 0.0),     # 8194 assignments: smallest chunked input
    (40000, 64, 2, 48, 1.1),    # 80000 assignments: chunked count / scan / scatter kernels
    (20001, 256, 6, 200, 0.5),  # ragged last chunk of the chunked kernels
]


@pytest.mark.parametrize("T,M,k,keep,skew", PERM_CASES)
def test_permute_is_bit_exact(T, M, k, keep, skew):
    say(f"permute T={T} M={M} k={k}")
    rng = np.random.default_rng(T * 31 + M)
    cand = sorted(rng.choice(M, keep, replace=False).tolist())
    idx, _ = W.gen_routing(T, M, k, cand, seed=T + M + k, skew=skew)
    d = 128
    x = rng.standard_normal((T, d)).astype(np.float32)
    xb = W.f32_to_bf16_bits(x)
    seg, src, inv, xp = E.permute(up_i32(idx), M, x=up(xb, W.BF16))
    rseg, rsrc, rinv = O.permute(idx, M)
    np.testing.assert_array_equal(down(seg), rseg)
    np.testing.assert_array_equal(down(src), rsrc)
    np.testing.assert_array_equal(down(inv), rinv)
    np.testing.assert_array_equal(down(xp), W.to_f64(xb, W.BF16)[rsrc])


def test_permute_without_gather_and_empty():
    idx = np.zeros((0, 2), np.int32)
    seg, src, inv, xp = E.permute(up_i32(idx), 8)
    assert down(seg).tolist() == [0] * 9 and xp is None


# ----------------------------------------------------------------------------- fixtures

class Layer:
    """Seeded inputs of one workload on host and device, with seeded routing."""

    def __init__(self, name, call_seed=None, **scale):
        cfg = name if isinstance(name, W.LayerConfig) else W.CONFIGS[name]
        cfg = cfg.scaled(**scale) if scale else cfg
        say(f"generating {cfg.name} T={cfg.n_tokens} d={cfg.d_model} M={cfg.n_experts} H={cfg.ffn_hidden}")
        self.cfg = cfg
        self.inp = W.gen_layer(cfg, call_seed=call_seed)
        cand = W.mask_members(self.inp.mask, cfg.n_experts)
        self.idx, self.w = W.gen_routing(cfg.n_tokens, cfg.n_experts, cfg.top_k, cand, seed=cfg.seed + 100,
                                         skew=cfg.zipf_s)
        dt = cfg.dtype
        self.x = up(self.inp.x, dt)
        self.wgu = up(self.inp.w_gate_up, dt)
        self.wdn = up(self.inp.w_down, dt)
        self.d_idx = up_i32(self.idx)
        self.d_w = up_f32(self.w)

    def expert_f64(self, e):
        return (W.to_f64(self.inp.w_gate_up[e], self.cfg.dtype), W.to_f64(self.inp.w_down[e], self.cfg.dtype))


_CACHE = {}


def layer(name, **scale):
    key = (name.name if isinstance(name, W.LayerConfig) else name, tuple(sorted(scale.items())))
    if key not in _CACHE:
        _CACHE.clear()
        torch.cuda.empty_cache()
        _CACHE[key] = Layer(name, **scale)
    return _CACHE[key]


# ----------------------------------------------------------------------------- experts + combine

@pytest.mark.parametrize("name", ["tiny", "small"])
def test_expert_ffn_and_moe_forward_full(name):
    L = layer(name)
    cfg = L.cfg
    seg, src, inv, _ = E.permute(L.d_idx, cfg.n_experts)
    y_perm, act = E.expert_ffn(L.x, seg, src, L.wgu, L.wdn, cfg.top_k, with_act=True)
    y = E.moe_forward(L.x, L.d_idx, L.d_w, L.wgu, L.wdn)
    torch.cuda.synchronize()
    x = L.inp.f64("x")
    gu = W.to_f64(L.inp.w_gate_up, cfg.dtype)
    dn = W.to_f64(L.inp.w_down, cfg.dtype)
    ry_perm, rseg, rsrc, rinv = O.expert_outputs(x, L.idx, gu, dn)
    # per-assignment outputs, each side through its own inverse permutation
    e1 = assert_close(down(y_perm)[down(inv)], ry_perm[rinv], tol(cfg.dtype), "y_perm")
    # the activation silu(gate) * up of every position, from the oracle's definition
    H = cfg.ffn_hidden
    ract = np.zeros((rsrc.size, H))
    for e in range(cfg.n_experts):
        lo, hi = rseg[e], rseg[e + 1]
        if hi > lo:
            h = x[rsrc[lo:hi]] @ gu[e].T
            ract[lo:hi] = O.silu(h[:, :H]) * h[:, H:]
    e2 = assert_close(down(act)[down(inv)], ract[rinv], tol(cfg.dtype), "act")
    ry = O.combine(ry_perm, rinv, L.w)
    e3 = assert_close(down(y), ry, tol(cfg.dtype), "y")
    say(f"  {name}: y_perm {e1:.2e} act {e2:.2e} y {e3:.2e}")


@pytest.mark.parametrize("name", ["mixtral", "finegrained", "decode"])
def test_moe_forward_full_size_every_row(name):
    """Full-size workload in the benchmark's launch configuration, compared on every row:
    the activation and the expert output of every assignment (each side through its own
    inverse permutation) and the combined output of every token. The oracle runs one
    expert segment at a time in float64 (weights upcast per expert)."""
    L = layer(name)
    cfg = L.cfg
    M, H = cfg.n_experts, cfg.ffn_hidden
    seg, src, inv, _ = E.permute(L.d_idx, M)
    y_perm, act = E.expert_ffn(L.x, seg, src, L.wgu, L.wdn, cfg.top_k, with_act=True)
    y = E.moe_forward(L.x, L.d_idx, L.d_w, L.wgu, L.wdn)
    torch.cuda.synchronize()
    rseg, rsrc, rinv = O.permute(L.idx, M)
    np.testing.assert_array_equal(down(seg), rseg)
    np.testing.assert_array_equal(down(src), rsrc)
    np.testing.assert_array_equal(down(inv), rinv)
    x = L.inp.f64("x")
    A = rsrc.size
    ract = np.zeros((A, H))
    ry_perm = np.zeros((A, cfg.d_model))
    for e in range(M):
        lo, hi = int(rseg[e]), int(rseg[e + 1])
        if hi == lo:
            continue
        gu, dn = L.expert_f64(e)
        h = x[rsrc[lo:hi]] @ gu.T
        ract[lo:hi] = O.silu(h[:, :H]) * h[:, H:]
        ry_perm[lo:hi] = O.swiglu_expert(x[rsrc[lo:hi]], gu, dn)
    # the same positions on both sides (the permutation is bit-exact): compare in place
    e_act = assert_close(down(act), ract, tol(cfg.dtype), "act")
    e_yp = assert_close(down(y_perm), ry_perm, tol(cfg.dtype), "y_perm")
    ry = O.combine(ry_perm, rinv, L.w)
    e_y = assert_close(down(y), ry, tol(cfg.dtype), "y")
    # every row on its own, relative to its own scale: no tile or split-K chunk may be off
    # while the tensor-wide figure still passes
    gy = down(y)
    row_err = np.max(np.abs(gy - ry), axis=1) / np.maximum(np.max(np.abs(ry), axis=1), 1e-30)
    assert np.max(row_err) <= 2 * tol(cfg.dtype), f"worst row {int(np.argmax(row_err))}: {np.max(row_err):.2e}"
    say(f"  {name}: act {e_act:.2e} y_perm {e_yp:.2e} y {e_y:.2e} (worst row {np.max(row_err):.2e}) over {A} "
        f"assignments, segments {np.diff(rseg).min()}..{np.diff(rseg).max()} rows")


@pytest.mark.parametrize("T,k,d,dt", [(777, 6, 2048, W.BF16),
                                      (5, 8, 4096, W.BF16),    # few tokens: rows split over workgroups
                                      (1, 2, 1024, W.BF16),
                                      (37, 3, 512, W.F32),
                                      (64, 16, 1024, W.F32),   # the widest slot count
                                      (50, 12, 768, W.BF16)])
def test_combine_matches_oracle(T, k, d, dt):
    rng = np.random.default_rng(21)
    idx, w = W.gen_routing(T, 64, k, range(64), seed=5)
    y32 = rng.standard_normal((T * k, d)).astype(np.float32)
    y_perm = W.f32_to_bf16_bits(y32) if dt == W.BF16 else y32
    _, _, rinv = O.permute(idx, 64)
    y = E.combine(up(y_perm, dt), up_i32(rinv), up_f32(w))
    ry = O.combine(W.to_f64(y_perm, dt), rinv, w)
    got = down(y)
    if dt == W.BF16:
        assert_close(got, ry, 2e-2, "combine")
        # a single rounding of a float32 sum: within one bfloat16 half-ulp plus float32 noise
        assert np.all(np.abs(got - ry) <= np.abs(ry) * 2.0 ** -8 + 1e-6)
    else:
        assert_close(got, ry, 1e-5, "combine")


def test_single_expert_layer_is_dense_ffn():
    """M = 1, k = 1: the MoE layer is the dense SwiGLU FFN of its one expert."""
    cfg = W.LayerConfig("dense", W.BF16, 300, 256, 1, 1, 384, 1, 16, 16, seed=9, mask="all", x_dist="rms")
    inp = W.gen_layer(cfg)
    idx = np.zeros((300, 1), np.int32)
    w = np.ones((300, 1), np.float32)
    y = E.moe_forward(up(inp.x, cfg.dtype), up_i32(idx), up_f32(w), up(inp.w_gate_up, cfg.dtype),
                      up(inp.w_down, cfg.dtype))
    ry = O.swiglu_expert(inp.f64("x"), W.to_f64(inp.w_gate_up[0], cfg.dtype), W.to_f64(inp.w_down[0], cfg.dtype))
    assert_close(down(y), ry, 2e-2, "dense")


def test_ragged_segments_and_empty_experts():
    """Segments far from tile multiples, experts with zero rows, tokens beyond one tile."""
    cfg = W.LayerConfig("ragged", W.BF16, 517, 256, 16, 4, 256, 3, 16, 16, seed=12, mask="random",
                        n_keep=5, x_dist="rms")
    inp = W.gen_layer(cfg)
    cand = W.mask_members(inp.mask, 16)
    idx, w = W.gen_routing(517, 16, 3, cand, seed=3, skew=1.5)
    y = E.moe_forward(up(inp.x, cfg.dtype), up_i32(idx), up_f32(w), up(inp.w_gate_up, cfg.dtype),
                      up(inp.w_down, cfg.dtype))
    ry = O.moe_forward(inp.f64("x"), idx, w, W.to_f64(inp.w_gate_up, cfg.dtype), W.to_f64(inp.w_down, cfg.dtype))
    assert_close(down(y), ry, 2e-2, "ragged")


def test_moe_forward_is_deterministic_and_needs_no_sync():
    L = layer("small")
    a = E.moe_forward(L.x, L.d_idx, L.d_w, L.wgu, L.wdn)
    b = E.moe_forward(L.x, L.d_idx, L.d_w, L.wgu, L.wdn)
    assert torch.equal(a, b)


def test_moe_forward_empty():
    L = layer("tiny")
    x = L.x[:0]
    y = E.moe_forward(x, L.d_idx[:0], L.d_w[:0], L.wgu, L.wdn)
    assert y.shape == (0, L.cfg.d_model)


@pytest.mark.parametrize("T,d,M,H,k,act,dt", [
    # experts of few rows take the streaming GEMM; rows a group (over all groups), tile:
    (1, 128, 8, 128, 2, "swiglu", W.BF16),     # 0: 32 x 128, fewer slabs than ring stages; 32 x 64
    (70, 256, 8, 2048, 1, "relu", W.BF16),     # 8: 32 x 64 in both layers
    (256, 128, 64, 1024, 1, "relu", W.BF16),   # 4: 32 x 128, then 32 x 64
    (1100, 128, 64, 1024, 1, "relu", W.BF16),  # 17: 64 x 128 with a second token tile in some groups, then 64 x 64
    (300, 384, 16, 640, 1, "swiglu", W.BF16),  # 18: 64 x 128, slabs no multiple of the ring
    (1400, 256, 16, 384, 1, "swiglu", W.BF16), # 87: 64 x 128 and 64 x 64 without the streaming policy
    (4480, 128, 64, 1024, 1, "relu", W.BF16),  # 70: 64 x 128 without it
    (9, 512, 8, 384, 1, "swiglu", W.F32),  # 1: 32 x 128 and 32 x 64 in float32
    (600, 384, 16, 640, 1, "relu", W.F32), # 37: 32 x 64 in float32
    (1000, 384, 8, 640, 1, "swiglu", W.F32),  # 125: 32 x 128, under a round of 64 x 128
    (1200, 128, 16, 640, 2, "swiglu", W.F32), # 150: 64 x 128
    (1200, 256, 16, 1152, 2, "relu", W.F32),  # 150: 32 x 128 without SwiGLU, K = 256
    (1200, 384, 16, 1536, 2, "relu", W.F32),  # 150: 32 x 64 over two rounds
])
def test_moe_forward_streaming_tiles(T, d, M, H, k, act, dt):
    cfg = W.LayerConfig("stream", dt, T, d, M, 1, H, k, min(T, 16), 16, seed=T, mask="all", x_dist="rms", activation=act)
    inp = W.gen_layer(cfg)
    cand = sorted(np.random.default_rng(T).choice(M, max(k, 3 * M // 4), replace=False).tolist())
    idx, w = W.gen_routing(T, M, k, cand, seed=T)
    y = E.moe_forward(up(inp.x, cfg.dtype), up_i32(idx), up_f32(w), up(inp.w_gate_up, cfg.dtype),
                      up(inp.w_down, cfg.dtype), activation=act)
    ry = O.moe_forward(inp.f64("x"), idx, w, W.to_f64(inp.w_gate_up, cfg.dtype), W.to_f64(inp.w_down, cfg.dtype), act)
    got = down(y)
    assert_close(got, ry, tol(dt), "y")
    row_err = np.max(np.abs(got - ry), axis=1) / np.maximum(np.max(np.abs(ry), axis=1), 1e-30)
    assert np.max(row_err) <= 2 * tol(dt), f"worst row {int(np.argmax(row_err))}: {np.max(row_err):.2e}"


@pytest.mark.parametrize("T,d,M,H,act,dt", [
    # rows a group over all groups, tile; the active groups have 0, 1, 2 and many token tiles:
    (900, 128, 64, 1024, "relu", W.BF16),    # 14: 32 x 128, then 32 x 64
    (1500, 256, 64, 384, "swiglu", W.BF16),  # 23: 64 x 128, slabs no multiple of the ring, then 64 x 64
    (900, 256, 8, 384, "relu", W.F32),       # 112: 32 x 64 in both layers, without the policy
    (900, 256, 64, 256, "swiglu", W.F32),    # 14: 32 x 128 in float32
])
def test_moe_forward_streaming_tiles_with_few_active_experts(T, d, M, H, act, dt):
    cfg = W.LayerConfig("masked", dt, T, d, M, 1, H, 1, 16, 16, seed=T, mask="all", x_dist="rms", activation=act)
    inp = W.gen_layer(cfg)
    # a group's rows: one, a tile's last row, one more, and the rest
    sizes = [1, 32, 33, 64, 65, T - 195]
    experts = np.linspace(0, M - 1, len(sizes)).astype(int)
    idx = np.random.default_rng(T).permutation(np.repeat(experts, sizes)).astype(np.int32)[:, None]
    w = np.random.default_rng(M).uniform(0.2, 1.0, (T, 1)).astype(np.float32)
    y = E.moe_forward(up(inp.x, cfg.dtype), up_i32(idx), up_f32(w), up(inp.w_gate_up, cfg.dtype),
                      up(inp.w_down, cfg.dtype), activation=act)
    ry = O.moe_forward(inp.f64("x"), idx, w, W.to_f64(inp.w_gate_up, cfg.dtype), W.to_f64(inp.w_down, cfg.dtype), act)
    got = down(y)
    assert_close(got, ry, tol(dt), "y")
    row_err = np.max(np.abs(got - ry), axis=1) / np.maximum(np.max(np.abs(ry), axis=1), 1e-30)
    assert np.max(row_err) <= 2 * tol(dt), f"worst row {int(np.argmax(row_err))}: {np.max(row_err):.2e}"


# ----------------------------------------------------------------------------- ReLU experts

def _relu_cfg(name, dtype, T, d, M, K, H, k, seed, n_keep=0):
    return W.LayerConfig(name, dtype, T, d, M, K, H, k, 16, 16, seed=seed,
                         mask="random" if n_keep else "all", n_keep=n_keep, x_dist="rms",
                         activation="relu")


RELU_FULL = [
    # every assignment against the oracle, activation included
    _relu_cfg("relu_f32", W.F32, 64, 128, 8, 2, 256, 2, seed=30, n_keep=6),   # fp32 register-staged GEMM
    _relu_cfg("relu_split", W.BF16, 64, 4096, 1, 1, 256, 1, seed=31),          # 2 tiles, K=4096: split-K reduce
    W.CONFIGS["switch8"],                                                     # paper shape, 3 candidates
    W.CONFIGS["switch64"],                                                    # paper shape, 25 candidates
]


@pytest.mark.parametrize("cfg", RELU_FULL, ids=lambda c: c.name)
def test_relu_expert_ffn_full(cfg):
    say(f"relu experts {cfg.name} T={cfg.n_tokens} d={cfg.d_model} M={cfg.n_experts} H={cfg.ffn_hidden}")
    L = layer(cfg)
    seg, src, inv, _ = E.permute(L.d_idx, cfg.n_experts)
    y_perm, act = E.expert_ffn(L.x, seg, src, L.wgu, L.wdn, cfg.top_k, with_act=True, activation="relu")
    y = E.moe_forward(L.x, L.d_idx, L.d_w, L.wgu, L.wdn, activation="relu")
    torch.cuda.synchronize()
    x = L.inp.f64("x")
    used = np.unique(L.idx)
    w_in = {int(e): W.to_f64(L.inp.w_gate_up[e], cfg.dtype) for e in used}
    dn = {int(e): W.to_f64(L.inp.w_down[e], cfg.dtype) for e in used}
    w_in_all = [w_in.get(e) for e in range(cfg.n_experts)]
    dn_all = [dn.get(e) for e in range(cfg.n_experts)]
    ry_perm, rseg, rsrc, rinv = O.expert_outputs(x, L.idx, w_in_all, dn_all, "relu")
    e1 = assert_close(down(y_perm)[down(inv)], ry_perm[rinv], tol(cfg.dtype), "y_perm")
    # relu(W_in x) of every position, from the definition
    ract = np.zeros((rsrc.size, cfg.ffn_hidden))
    for e in used:
        lo, hi = rseg[e], rseg[e + 1]
        ract[lo:hi] = np.maximum(x[rsrc[lo:hi]] @ w_in[int(e)].T, 0.0)
    got_act = down(act)
    assert np.all(got_act >= 0.0), "ReLU activation has negative entries"
    e2 = assert_close(got_act[down(inv)], ract[rinv], tol(cfg.dtype), "act")
    ry = O.combine(ry_perm, rinv, L.w)
    e3 = assert_close(down(y), ry, tol(cfg.dtype), "y")
    say(f"  {cfg.name}: y_perm {e1:.2e} act {e2:.2e} y {e3:.2e}")


def test_relu_moe_forward_large_tiles_every_row():
    """Enough rows per expert for the 256x256 ping-pong GEMM and its split-K tail, with
    the ReLU applied in the staged epilogue; every row against the oracle."""
    cfg = _relu_cfg("relu_big", W.BF16, 8192, 1024, 8, 2, 2048, 1, seed=32)
    L = layer(cfg)
    y = E.moe_forward(L.x, L.d_idx, L.d_w, L.wgu, L.wdn, activation="relu")
    torch.cuda.synchronize()
    x = L.inp.f64("x")
    w_in = [W.to_f64(L.inp.w_gate_up[e], cfg.dtype) for e in range(cfg.n_experts)]
    dn = [W.to_f64(L.inp.w_down[e], cfg.dtype) for e in range(cfg.n_experts)]
    ry = O.moe_forward(x, L.idx, L.w, w_in, dn, "relu")
    e = assert_close(down(y), ry, tol(cfg.dtype), "y")
    say(f"  relu_big: y rel err {e:.2e} over {cfg.n_tokens} tokens")


def test_relu_and_swiglu_weights_are_not_interchangeable():
    """The binding checks the input-layer weight shape against the activation."""
    L = layer(W.CONFIGS["switch8"])
    with pytest.raises(ValueError):
        E.moe_forward(L.x, L.d_idx, L.d_w, L.wgu, L.wdn, activation="swiglu")
