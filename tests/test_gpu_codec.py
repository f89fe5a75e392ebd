"""Parity of the low-rank encoder/decoder kernels with the oracle
(Encoder-Decoder based on Low-Rank Compression: Z = U^T X V, X_hat = U_hat Z V_hat^T)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2508_06024_amd import ec2moe as E
from paper_2508_06024_amd import workload as W
from tests.gpu_common import TOL_F32, assert_close, down, say, tol, up, up_f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", W.CONFIG_ORDER)
def test_codec_matches_oracle_at_full_size(name):
    cfg = W.CONFIGS[name]
    say(f"codec {name}: h={cfg.n_tokens} w={cfg.d_model} r_h={cfg.r_h} r_w={cfg.r_w}")
    inp = W.gen_layer(cfg, experts=False)
    x, u, v = (up(getattr(inp, n), cfg.dtype) for n in ("x", "u", "v"))
    z = E.lowrank_encode(x, u, v)
    xh = E.lowrank_decode(z, u, v)
    torch.cuda.synchronize()
    rz = O.lowrank_encode(inp.f64("x"), inp.f64("u"), inp.f64("v"))
    rxh = O.lowrank_decode(rz, inp.f64("u"), inp.f64("v"))
    ez = assert_close(down(z), rz, TOL_F32, "Z")
    exh = assert_close(down(xh), rxh, tol(cfg.dtype), "X_hat")
    say(f"  Z {ez:.2e}  X_hat {exh:.2e}")


def test_full_rank_codec_round_trips_on_gpu():
    """Square orthogonal U, V (the tiny workload's T=64, d=128 at full rank... r <= 256):
    decode(encode(X)) = X within float32 rounding."""
    cfg = W.CONFIGS["tiny"]
    x = W.gen_call(cfg)[0]
    u = W.haar_orthonormal(5, (1,), 64, 64).astype(np.float32)
    v = W.haar_orthonormal(5, (2,), 128, 128).astype(np.float32)
    z = E.lowrank_encode(up(x, W.F32), up(u, W.F32), up(v, W.F32))
    xh = E.lowrank_decode(z, up(u, W.F32), up(v, W.F32))
    assert_close(down(xh), x.astype(np.float64), 1e-5, "round trip")


@pytest.mark.parametrize("c,h,w,rh,rw,dt", [
    (2, 300, 384, 32, 48, W.BF16),
    (5, 64, 256, 16, 32, W.F32),
    (17, 40, 128, 16, 16, W.BF16),   # more slices than one batch of launches (16)
    (4, 256, 768, 64, 64, W.BF16),   # the paper-shaped layers: 4 sequences of 256 tokens
    (1, 300, 256, 80, 64, W.BF16),   # r_h ending inside the second 64-row block of U^T P
    (2, 260, 128, 208, 112, W.F32),  # ... inside the fourth
    # float32 products with K in no whole 512-byte slabs, dense and grouped
    (1, 300, 512, 48, 48, W.F32),
    (2, 200, 512, 96, 160, W.F32),
    (4, 100, 512, 32, 32, W.F32),
    (3, 90, 256, 80, 16, W.F32),
    # bf16 layers take the fused encoder, here in whole 64-token, 64-column tiles:
    (3, 128, 256, 80, 128, W.BF16),   # r_h inside the second 64-row block, two column tiles
    (2, 256, 384, 256, 192, W.BF16),  # three column tiles of a token tile placed on one XCD
    (17, 128, 128, 16, 64, W.BF16),   # two tiles per slice, more slices than one batch
    # the decoder's expansion kernel in whole 128-token bands:
    (1, 128, 128, 128, 64, W.BF16),    # one band of two 64-column chunks
    (1, 256, 512, 256, 128, W.BF16),   # with the fused encoder
    (1, 4000, 2176, 48, 32, W.BF16),   # runs of three chunks, a ragged last band, rank padded to 64
    (3, 129, 256, 64, 256, W.BF16),    # one launch, the largest r_w, one token in the second band
    (1, 200, 384, 112, 112, W.BF16),   # one launch with padded ranks of 128
    (1, 4096, 2176, 128, 64, W.BF16),  # runs of three chunks, the last of each band one chunk (34 chunks)
    (2, 256, 384, 32, 48, W.BF16),     # one launch, whole bands, rank 32
    (3, 520, 2304, 64, 256, W.BF16),   # ... five bands, the largest r_w, ragged
    (1, 3968, 2304, 64, 256, W.BF16),  # ... whole bands, runs of three chunks
    # two launches with a ragged last band and several chunks a workgroup:
    (1, 4001, 2176, 128, 64, W.BF16),
    (2, 2001, 2176, 256, 208, W.BF16),
    (1, 4001, 2176, 144, 256, W.BF16),  # rank padded to 256
    # ... with a last tile of one token or column block, and the width in shares of unequal stages:
    (1, 65, 1152, 64, 16, W.BF16),     # 9 stages in 4 shares, one token in the second tile
    (1, 127, 128, 16, 80, W.BF16),     # one stage
    (2, 1000, 640, 144, 208, W.BF16),  # tiles of two slices in one share
    # ... and many token tiles with large partial sums, in runs whose sums stay in registers:
    (1, 20001, 128, 128, 128, W.BF16),  # 313 tiles in 128 runs of two or three, 33 tokens in the last
    (2, 8193, 256, 144, 208, W.BF16),   # 129 tiles in 32 runs of two slices, one token in the last
    (17, 2100, 128, 128, 80, W.BF16),   # 33 tiles in 8 runs; the second batch has a single slice
    # at most 64 tokens per slice take the small-batch encoder and decoder:
    (3, 48, 256, 32, 48, W.BF16),
    (2, 64, 256, 64, 256, W.F32),     # the largest r_h and r_w of that path
])
def test_codec_slices_and_separate_decoder_projections(c, h, w, rh, rw, dt):
    """Several slices coded with one U, V; decoder projections different from the encoder's."""
    say(f"codec slices c={c} h={h} w={w} r={rh}x{rw} {dt}")
    rng = np.random.default_rng(3 + c)
    cast = (lambda a: W.f32_to_bf16_bits(np.asarray(a, np.float32))) if dt == W.BF16 else (lambda a: np.asarray(a, np.float32))
    x = cast(rng.standard_normal((c, h, w)))
    u = cast(W.haar_orthonormal(1, (1,), h, rh))
    v = cast(W.haar_orthonormal(1, (2,), w, rw))
    uh = cast(rng.standard_normal((h, rh)) * 0.1)
    vh = cast(rng.standard_normal((w, rw)) * 0.1)
    z = E.lowrank_encode(up(x, dt), up(u, dt), up(v, dt))
    xh = E.lowrank_decode(z, up(uh, dt), up(vh, dt))
    f = lambda a: W.to_f64(a, dt)
    for s in range(c):
        rz = O.lowrank_encode(f(x[s]), f(u), f(v))
        assert_close(down(z[s]), rz, TOL_F32, f"Z[{s}]")
        assert_close(down(xh[s]), O.lowrank_decode(rz, f(uh), f(vh)), tol(dt), f"X_hat[{s}]")


@pytest.mark.parametrize("c,h,w,rh,rw", [
    (1, 130, 256, 16, 32),    # one launch, rank padded to 32
    (2, 130, 256, 48, 64),    # ... to 64
    (1, 200, 384, 112, 112),  # ... to 128
    (1, 150, 256, 144, 64),   # two launches, rank padded to 256
])
def test_infinity_in_a_padded_rank_reaches_only_its_own_column(c, h, w, rh, rw):
    """An infinite projection value of one model column: with positive factors that column of X_hat is
    +inf in every token, and every other column is finite."""
    rng = np.random.default_rng(rh)
    pos = lambda *shape: W.f32_to_bf16_bits(rng.uniform(0.5, 1.0, shape).astype(np.float32))
    uh, vh = pos(h, rh), pos(w, rw)
    vh[w // 2, rw // 3] = 0x7F80
    z = rng.uniform(0.5, 1.0, (c, rh, rw)).astype(np.float32)
    got = down(E.lowrank_decode(up_f32(z), up(uh, W.BF16), up(vh, W.BF16)))
    hit = np.arange(w) == w // 2
    assert np.all(np.isposinf(got[..., hit]))
    assert np.all(np.isfinite(got[..., ~hit]))


def test_codec_is_deterministic():
    cfg = W.CONFIGS["small"]
    inp = W.gen_layer(cfg, experts=False)
    x, u, v = (up(getattr(inp, n), cfg.dtype) for n in ("x", "u", "v"))
    z1, z2 = E.lowrank_encode(x, u, v), E.lowrank_encode(x, u, v)
    assert torch.equal(z1, z2)
    assert torch.equal(E.lowrank_decode(z1, u, v), E.lowrank_decode(z2, u, v))
