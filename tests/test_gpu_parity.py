"""GPU parity: every C-ABI entry point against the CPU oracle, element by element, on the
same seeded inputs.  Integer outputs (expert indices, offsets, permutations) must be
bit-exact; fp32 outputs within 1e-4 relative, bf16 outputs within 2e-2 relative
(per-tensor max-abs and L2 relative error, whichever is larger).

Routing on random inputs: the GPU sums logits in fp32, the oracle in fp64, so a token
whose k-th and (k+1)-th logits are closer than the fp32 rounding bound of the dot product
is "ambiguous"; indices must match exactly on every other token, and on ambiguous ones
the GPU's choice must still be admissible.  Tie-break tests use inputs whose fp32 dot
products are exact in any order, so equality there is genuinely bit-exact.
"""
import numpy as np
import pytest
import torch

import paper_2503_00245_amd as pkg
import workloads as wl
from tests.helpers import (ambiguous_tokens, bits_of, elementwise_rel_err, rel_err, row_rel_err,
                           stored_f64, to_device, to_f64, weights_to_device)

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}
# Worst element-wise relative error over the elements above a tenth of the tensor's rms.  bf16: the
# path rounds the hidden tensor, the grouped output rows and the result to bf16 (2^-9 relative
# each, independent), which leaves an absolute error of about 1.5e-3 rms per element, 5 sigma
# = 8e-3 rms over millions of elements, i.e. 0.08 relative at the magnitude floor; the bound
# leaves a factor 2.5.  fp32: fp32 accumulation over a few thousand terms, about 1e-6 rms.
ELEMENTWISE_TOL = {"f32": 1e-3, "bf16": 0.2}
DT = {"f32": pkg.MOE_F32, "bf16": pkg.MOE_BF16}


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pkg.lib()  # fail loudly if the HIP library is not built
    return torch.device("cuda:0")


def _cfg(name="t", d=128, F=256, E=4, k=2, dtype="bf16", seed=1, r=0, base=False, std=0.02):
    return wl.LayerConfig(name, d, F, E, k, dtype, seed, rank=r, shared_base=base,
                          weight_std=std, wd_product_std=std if not base else std / 4)


def _check_routing(oracle, x_np, w_np, k, idx_gpu, gate_gpu, probs_gpu=None):
    """Bit-exact indices off the ambiguous set; gates/probs to fp32 accuracy. Returns mask of
    tokens whose routing equals the oracle's."""
    idx, gate, probs, logits = oracle.route(x_np, w_np["router_w"], w_np["router_b"], k)
    amb = ambiguous_tokens(logits, x_np, w_np["router_w"], k)
    same = np.all(idx_gpu == idx, axis=1)
    assert np.all(same[~amb]), f"routing differs on {int((~same & ~amb).sum())} unambiguous tokens"
    # an ambiguous token may pick differently, but only experts within the rounding band
    for t in np.flatnonzero(~same):
        kth = np.sort(logits[t])[::-1][k - 1]
        assert len(set(idx_gpu[t])) == k
        assert np.all(logits[t, idx_gpu[t]] >= kth - 1e-4), "inadmissible choice on ambiguous token"
    # k + 1 adjacent ranks can each be a near-tie, so the allowance grows with k
    assert amb.sum() <= max(2, x_np.shape[0] * k // 400), "too many ambiguous tokens for this recipe"
    assert np.allclose(gate_gpu[same], gate[same], rtol=2e-5, atol=1e-7)
    assert np.allclose(gate_gpu.sum(1), 1.0, atol=1e-6)
    if probs_gpu is not None:
        assert np.allclose(probs_gpu, probs, rtol=2e-5, atol=1e-8)
    return same, idx, gate


def _route_gpu(dev, x_t, w_t, E, k, act, want_probs=True):
    T, d = x_t.shape
    shape = pkg.make_shape(T, d, 8, E, k, 0, act)
    idx = torch.full((T, k), -7, dtype=torch.int32, device=dev)
    gate = torch.full((T, k), -7.0, dtype=torch.float32, device=dev)
    probs = torch.full((T, E), -7.0, dtype=torch.float32, device=dev) if want_probs else None
    pkg.moe_route(shape, x_t, w_t["router_w"], w_t["router_b"], idx, gate, probs)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), gate.cpu().numpy().astype(np.float64), \
        None if probs is None else probs.cpu().numpy().astype(np.float64)


# ------------------------------------------------------------------------------- moe_route

@pytest.mark.parametrize("T,d,E,k,dtype,bias", [
    (32, 128, 4, 2, "f32", False),      # tiny config
    (77, 1024, 8, 2, "bf16", False),    # wearables width, ragged token count
    (300, 2048, 8, 2, "bf16", True),    # phone width with a router bias
    (1, 2048, 8, 2, "bf16", True),      # single-token decode
    (65, 256, 64, 8, "bf16", True),     # one expert per lane
    (33, 264, 5, 1, "f32", False),      # k = 1, d not a multiple of the wave stride
    (40, 512, 6, 6, "bf16", False),     # k = E
    (19, 128, 64, 64, "bf16", True),    # the largest E and k the library takes
    (1500, 1024, 8, 2, "bf16", True),   # many tokens: eight per workgroup, ragged last tile
    (1028, 256, 64, 8, "f32", False),
    (2048, 2048, 8, 2, "bf16", True),   # phone prefill
    # 8192 tokens and more with at most 16 experts: the kernel that stages the router in LDS
    (8200, 2048, 8, 2, "bf16", True),   # phone width, three tokens per wave, ragged token count
    (8192, 264, 5, 1, "f32", False),    # d not a multiple of the wave stride
    (8192, 2048, 16, 4, "bf16", False), # the largest router that fits (128 KB)
    (20000, 512, 8, 8, "bf16", True),   # five tokens per wave, k = E
])
def test_route_matches_oracle(dev, oracle, T, d, E, k, dtype, bias):
    cfg = _cfg(d=d, E=E, k=k, dtype=dtype, seed=300 + T)
    w_np = wl.make_layer_weights(cfg, with_bias=False)
    if bias:
        w_np["router_b"] = wl.normal_tensor(cfg.seed, 99, (E,), 0.5, "f32")
    x_np = wl.make_inputs(cfg, T)
    w_t = weights_to_device({"router_w": w_np["router_w"], "router_b": w_np["router_b"]}, dev)
    idx, gate, probs = _route_gpu(dev, to_device(x_np, dev), w_t, E, k, DT[dtype])
    _check_routing(oracle, x_np, w_np, k, idx, gate, probs)
    if k == 1:
        assert np.all(gate == 1.0)


def test_route_large_batch_kernel_is_bit_identical_to_the_small_batch_one(dev):
    # the same tokens routed as one batch of 9000 (router staged in LDS, wave per token) and in
    # slices of 3000 (wave per expert): logits are summed in the same order, so every output
    # matches bit for bit
    cfg = _cfg(d=1024, E=8, k=2, dtype="bf16", seed=321)
    w_np = wl.make_layer_weights(cfg, with_bias=False)
    w_np["router_b"] = wl.normal_tensor(cfg.seed, 99, (8,), 0.5, "f32")
    x_np = wl.make_inputs(cfg, 9000)
    w_t = weights_to_device({"router_w": w_np["router_w"], "router_b": w_np["router_b"]}, dev)
    idx, gate, probs = _route_gpu(dev, to_device(x_np, dev), w_t, 8, 2, pkg.MOE_BF16)
    for lo in range(0, 9000, 3000):
        i2, g2, p2 = _route_gpu(dev, to_device(np.ascontiguousarray(x_np[lo:lo + 3000]), dev), w_t, 8, 2,
                                pkg.MOE_BF16)
        assert np.array_equal(idx[lo:lo + 3000], i2)
        assert np.array_equal(gate[lo:lo + 3000], g2) and np.array_equal(probs[lo:lo + 3000], p2)


@pytest.mark.parametrize("T", [512, 8704])
def test_route_tie_break_is_lowest_index_bit_exact(dev, oracle, T):
    # entries in {-1, -.5, 0, .5, 1} and a 0/1 router: every partial sum is exact in fp32
    rng = np.random.default_rng(5)
    E, d, k = 8, 64, 3
    x = (rng.integers(-2, 3, size=(T, d)) * 0.5).astype(np.float32)
    rw = np.zeros((E, d), np.float32)
    for e in range(E):
        rw[e, rng.choice(d, size=4, replace=False)] = 1.0
    rw[5] = rw[2]          # duplicated router rows: permanent ties between experts 2 and 5
    rw[7] = rw[0]
    w_np = {"router_w": rw, "router_b": None}
    for dtype in ("f32", "bf16"):
        x_np = x if dtype == "f32" else wl.f32_to_bf16_bits(x)
        idx, gate, _ = _route_gpu(dev, to_device(x_np, dev), weights_to_device(w_np, dev), E, k,
                                  DT[dtype])
        ref_idx, ref_gate, _, logits = oracle.route(x_np, rw, None, k)
        assert np.array_equal(idx, ref_idx)
        assert np.allclose(gate, ref_gate, rtol=1e-5)
        assert (np.sort(logits, 1)[:, -k] == np.sort(logits, 1)[:, -k - 1]).sum() > 20  # ties at the cut
    # all-zero router: every logit equal -> experts 0..k-1, gates exactly 1/k when k is a power of 2
    z = {"router_w": np.zeros((E, d), np.float32), "router_b": None}
    idx, gate, probs = _route_gpu(dev, to_device(x, dev), weights_to_device(z, dev), E, 2, pkg.MOE_F32)
    assert np.array_equal(idx, np.tile(np.arange(2, dtype=np.int32), (T, 1)))
    assert np.all(gate == 0.5) and np.all(probs == 0.125)


# ------------------------------------------------------------------------------- moe_permute

@pytest.mark.parametrize("T,k,E", [(1, 1, 1), (1, 2, 8), (37, 2, 4), (512, 2, 8), (2048, 2, 8),
                                   (4096, 2, 8), (4097, 2, 8), (1000, 8, 64), (50000, 3, 7)])
def test_permute_matches_oracle_bit_exact(dev, oracle, T, k, E):
    rng = np.random.default_rng(T * 31 + E)
    # k distinct experts per token, skewed so some experts are empty or tiny
    scores = rng.standard_normal((T, E)) + np.linspace(2, -2, E)
    if E > 2:
        scores[:, 1] = -100  # expert 1 never chosen
    keys = np.argsort(-scores, axis=1)[:, :k].astype(np.int32)
    d = 64
    x_np = wl.normal_tensor(T, 1, (T, d), 1.0, "bf16")
    shape = pkg.make_shape(T, d, 64, E, k, 0, pkg.MOE_BF16)
    P = T * k
    off = torch.full((E + 1,), -1, dtype=torch.int32, device=dev)
    perm = torch.full((P,), -1, dtype=torch.int32, device=dev)
    inv = torch.full((P,), -1, dtype=torch.int32, device=dev)
    x_t = to_device(x_np, dev)
    xp = torch.zeros((P, d), dtype=torch.bfloat16, device=dev)
    ws = pkg.alloc_workspace(shape, dev)
    pkg.moe_permute(shape, to_device(keys, dev), off, perm, inv, x_t, xp, ws)
    torch.cuda.synchronize()
    r_off, r_perm, r_inv = oracle.permute(keys, E)
    assert np.array_equal(off.cpu().numpy(), r_off)
    assert np.array_equal(perm.cpu().numpy(), r_perm)
    assert np.array_equal(inv.cpu().numpy(), r_inv)
    assert np.array_equal(bits_of(xp), x_np[r_perm // k])
    # unpermute(permute(x)) is the identity on the payload
    assert np.array_equal(bits_of(xp)[r_inv].reshape(T, k, d)[:, 0], x_np)


@pytest.mark.parametrize("T,k,E,room", [
    # one pair more than a workgroup sorts alone; a last chunk of one pair; 256 chunks and the first size past them; many experts
    (8193, 1, 3, 1 << 20), (5121, 2, 8, 1 << 20), (65536, 4, 16, 1 << 20), (65537, 4, 16, 1 << 20), (9000, 3, 64, 1 << 20),
    (5121, 2, 8, None), (65537, 4, 16, None),  # no more scratch than is asked for: longer chunks
])
def test_permute_in_chunks_of_any_length(dev, oracle, T, k, E, room):
    rng = np.random.default_rng(T + E)
    keys = np.sort(rng.integers(0, E, (T, k)), axis=1).astype(np.int32)  # (the sort takes repeated experts, too)
    keys[: T // 3] = rng.integers(0, max(1, E // 4), (T // 3, k))
    shape = pkg.make_shape(T, 8, 8, E, k, 0, pkg.MOE_BF16)
    need = ((T * k + 8191) // 8192 * E * 4 + 255) // 256 * 256
    off, perm, inv = (torch.full((n,), -1, dtype=torch.int32, device=dev) for n in (E + 1, T * k, T * k))
    ws = torch.empty(room or need, dtype=torch.uint8, device=dev)
    pkg.moe_permute(shape, to_device(keys, dev), off, perm, inv, None, None, ws)
    torch.cuda.synchronize()
    for got, ref in zip((off, perm, inv), oracle.permute(keys, E)):
        assert np.array_equal(got.cpu().numpy(), ref)


@pytest.mark.parametrize("T,d,E,k,dtype", [
    (8192, 72, 5, 2, "bf16"), (16385, 520, 8, 3, "bf16"), (8193, 1032, 9, 1, "bf16"), (12289, 264, 16, 4, "bf16"), (8195, 68 * 4, 7, 2, "f32"),
    (12290, 520, 12, 2, "bf16"), (20483, 72, 10, 3, "f32"), (12287, 136, 16, 2, "bf16"), (12291, 1032, 13, 2, "bf16"),
])
def test_route_several_tokens_per_wave(dev, oracle, T, d, E, k, dtype):
    # two, three and four tokens at a time, remainders of a wave's share, ragged chunks, up to 8, 12 and 16 experts
    cfg = _cfg(d=d, F=8, E=E, k=k, dtype=dtype, seed=2100 + T + E)
    w_np = wl.make_layer_weights(cfg)
    x_np = wl.make_inputs(cfg, T)
    idx, gate, probs = _route_gpu(dev, to_device(x_np, dev), weights_to_device(w_np, dev), E, k, DT[dtype])
    _check_routing(oracle, x_np, w_np, k, idx, gate, probs)


@pytest.mark.parametrize("T,k,E", [(1_000_000, 4, 64), ((1 << 21) - 1, 8, 8)])
def test_permute_large_without_payload(dev, oracle, T, k, E):
    # several hundred workgroups per kernel of the multi-pass sort; the second case is the
    # largest pair count the library accepts (T k just under 2^24)
    rng = np.random.default_rng(E * 1000 + k)
    keys = np.argsort(rng.random((T, E), dtype=np.float32) + np.linspace(0.6, 0, E, dtype=np.float32),
                      axis=1)[:, :k].astype(np.int32)
    shape = pkg.make_shape(T, 8, 8, E, k, 0, pkg.MOE_BF16)
    P = T * k
    assert P < (1 << 24)
    off = torch.full((E + 1,), -1, dtype=torch.int32, device=dev)
    perm = torch.full((P,), -1, dtype=torch.int32, device=dev)
    inv = torch.full((P,), -1, dtype=torch.int32, device=dev)
    ws = pkg.alloc_workspace(shape, dev)
    pkg.moe_permute(shape, to_device(keys, dev), off, perm, inv, None, None, ws)
    torch.cuda.synchronize()
    r_off, r_perm, r_inv = oracle.permute(keys, E)
    assert np.array_equal(off.cpu().numpy(), r_off)
    assert np.array_equal(perm.cpu().numpy(), r_perm)
    assert np.array_equal(inv.cpu().numpy(), r_inv)


# ------------------------------------------------------------------------------- moe_expert_ffn

def _ffn_case(dev, oracle, cfg, offsets, tol):
    w_np = wl.make_layer_weights(cfg, with_bias=False)
    P = int(offsets[-1])
    xp_np = wl.normal_tensor(cfg.seed, 77, (P, cfg.d_model), 1.0, cfg.act_dtype)
    w_t = weights_to_device(w_np, dev)
    # the staged call sees P rows as P "tokens" with k = 1
    shape = pkg.shape_for(w_t, P, 1, DT[cfg.act_dtype])
    ws = pkg.alloc_workspace(shape, dev)
    xp = to_device(xp_np, dev)
    yp = torch.full_like(xp, float("nan"))
    pkg.moe_expert_ffn(shape, pkg.make_weights(w_t), xp, to_device(offsets, dev), yp, ws)
    torch.cuda.synchronize()
    ref = oracle.expert_ffn(w_np, xp_np, offsets)
    got = to_f64(yp)
    assert np.all(np.isfinite(got))
    err = rel_err(got, ref)
    assert err < tol, f"relative error {err:.3e} >= {tol}"
    return err


def test_expert_ffn_tiny_fp32(dev, oracle):
    cfg = _cfg(d=128, F=256, E=4, dtype="f32", seed=401, std=0.05)
    _ffn_case(dev, oracle, cfg, np.array([0, 20, 20, 49, 64], np.int32), TOL["f32"])


@pytest.mark.parametrize("d,F,offsets", [
    (256, 384, [0, 130, 130, 257, 300]),          # several m-tiles, an empty expert, ragged tails
    (200, 328, [0, 1, 3, 70, 71]),                # K and N not multiples of the tile, tiny groups
    (1024, 2816, [0, 64, 200, 200, 333, 333, 400, 401, 520]),  # wearables widths, 8 experts
    # 585 gate/up tiles of 256 x 256: 74 (or 67) per XCD = two rounds of 32 and a thin third one, whose
    # tiles are cut into upper and lower halves; the cut tiles include ragged ones (164 and 120 live rows)
    (128, 5760, [0, 1700, 3100]),
    # 540 gate/up tiles of 256 x 256: 68 per XCD = two rounds and 4 tiles that are cut
    (128, 5760, [0, 1700, 2900]),
    # the same for a kernel that runs two workgroups per CU: 576 down tiles of 128 x 128, 72 per XCD =
    # one round of 64 and 8 tiles cut into halves (the last tile of the second group holds 74 rows)
    (2048, 192, [0, 2304, 4554]),
    # K tails in the 256-row kernel: K = 72 is two k-steps of 32 and a tail of 8; the down product
    # then has K = 4008 (a tail of 40 in a 64-wide step)
    (72, 4008, [0, 1700, 3100]),
    # K shorter than one k-step: the only step is the tail
    (24, 4104, [0, 1500, 3000]),
])
def test_expert_ffn_dense_bf16(dev, oracle, d, F, offsets):
    cfg = _cfg(d=d, F=F, E=len(offsets) - 1, dtype="bf16", seed=402 + d, std=0.05)
    _ffn_case(dev, oracle, cfg, np.array(offsets, np.int32), TOL["bf16"])


# as many tiles as the rows can need: one row past whole tiles of 64, 128 and 256 rows in every group
@pytest.mark.parametrize("d,F,dtype,loads", [
    (256, 384, "bf16", [257, 1, 513, 1, 1, 257, 1, 1]), (256, 2048, "bf16", [129] * 5 + [1] * 3), (128, 704, "bf16", [65] * 16),
    (256, 5760, "bf16", [1537, 1]), (64, 128, "f32", [17, 33, 1, 49]),
])
def test_expert_ffn_at_the_bound_of_tiles(dev, oracle, d, F, dtype, loads):
    cfg = _cfg(d=d, F=F, E=len(loads), dtype=dtype, seed=431 + d, std=0.05)
    _ffn_case(dev, oracle, cfg, np.cumsum([0] + loads).astype(np.int32), TOL[dtype])


@pytest.mark.parametrize("d,F,r,offsets", [
    # gate/up products on 256-row tiles (two experts, 45 column tiles): one, two, three k-steps, tails of 8, 56
    # and 8 columns, groups that end 1 and 255 rows into a tile
    (64, 5760, 0, [0, 1537, 3072]), (72, 5760, 0, [0, 1537, 3072]), (120, 5760, 0, [0, 1700, 3100]),
    (136, 5760, 0, [0, 1791, 3100]), (192, 5768, 0, [0, 1700, 3100]),
    # plain products on them: 8192 and 8200 columns (a last column tile of 8), K of 72 and 200
    (8192, 72, 0, [0, 1537, 3100]), (8200, 200, 0, [0, 1700, 3100]),
    # two activation operands: K of one, one and a bit, and several k-steps, each walked twice
    (128, 5760, 64, [0, 1537, 3072]), (128, 5760, 72, [0, 1700, 3100]), (128, 5760, 200, [0, 1791, 3100]),
])
def test_expert_ffn_on_256_row_tiles(dev, oracle, d, F, r, offsets):
    cfg = _cfg(d=d, F=F, E=len(offsets) - 1, dtype="bf16", seed=430 + d + r, r=r, std=0.05)
    _ffn_case(dev, oracle, cfg, np.array(offsets, np.int32), TOL["bf16"])


@pytest.mark.parametrize("d,F,r,offsets", [
    # few rows per group (64- and 128-row tiles): single rows, 63 / 64 / 65 rows, an empty expert; K of one k-step,
    # fewer steps than LDS holds, a tail; widths fitted to 256 workgroups down to 8 columns
    (64, 264, 0, [0, 1, 1, 3, 4]), (136, 520, 0, [0, 63, 127, 192, 193]), (320, 1000, 0, [0, 64, 64, 129, 200]),
    (200, 72, 0, [0, 96, 97, 160, 250]), (1024, 2816, 0, [0, 5, 9, 70, 71]),
    (256, 448, 64, [0, 1, 65, 65, 70]), (200, 328, 104, [0, 40, 104, 169, 240]), (640, 640, 72, [0, 128, 256, 385, 400]),
])
def test_expert_ffn_on_small_tiles(dev, oracle, d, F, r, offsets):
    cfg = _cfg(d=d, F=F, E=len(offsets) - 1, dtype="bf16", seed=460 + d + r, r=r, std=0.05)
    _ffn_case(dev, oracle, cfg, np.array(offsets, np.int32), TOL["bf16"])


@pytest.mark.parametrize("d,F,r,base,T", [
    (256, 2120, 104, False, 5), (256, 2120, 104, False, 130), (512, 4104, 256, False, 300),  # rank-down in fp32 parts
    (256, 2120, 64, True, 3), (264, 4104, 40, True, 90), (512, 2816, 64, True, 700),         # and the base's down
])
def test_forward_products_cut_along_k(dev, oracle, d, F, r, base, T):
    cfg = _cfg(d=d, F=F, E=8, dtype="bf16", seed=480 + d + T, r=r, base=base, std=0.05)
    _forward_case(dev, oracle, cfg, T)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("base", [False, True])
def test_expert_ffn_weight_decomposed(dev, oracle, dtype, base):
    cfg = _cfg(d=256, F=448, E=4, dtype=dtype, seed=410, r=(40 if base else 128), base=base, std=0.05)
    _ffn_case(dev, oracle, cfg, np.array([0, 150, 150, 161, 300], np.int32), TOL[dtype])


# ------------------------------------------------------------------------------- moe_combine

@pytest.mark.parametrize("dtype,residual", [("f32", False), ("bf16", True), ("bf16", False)])
def test_combine_matches_oracle(dev, oracle, dtype, residual):
    T, k, d, E = 75, 3, 264, 6
    rng = np.random.default_rng(9)
    keys = np.argsort(rng.standard_normal((T, E)), axis=1)[:, :k].astype(np.int32)
    _, _, inv = oracle.permute(keys, E)
    yp_np = wl.normal_tensor(9, 1, (T * k, d), 1.0, dtype)
    res_np = wl.normal_tensor(9, 2, (T, d), 1.0, dtype) if residual else None
    g = rng.random((T, k)).astype(np.float32)
    g /= g.sum(1, keepdims=True)
    shape = pkg.make_shape(T, d, 64, E, k, 0, DT[dtype])
    y = torch.empty((T, d), dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device=dev)
    pkg.moe_combine(shape, to_device(yp_np, dev), to_device(inv, dev), to_device(g, dev),
                    to_device(res_np, dev), y)
    torch.cuda.synchronize()
    ref = oracle.combine(stored_f64(yp_np), inv, g.astype(np.float64), residual=res_np)
    assert rel_err(to_f64(y), ref) < (1e-6 if dtype == "f32" else 5e-3)


# ------------------------------------------------------------------------------- moe_forward

def _forward_gpu(dev, w_t, x_t, k, act, residual=False):
    T = x_t.shape[0]
    shape = pkg.shape_for(w_t, T, k, act, residual=residual)
    ws = pkg.alloc_workspace(shape, dev)
    y = torch.full_like(x_t, float("nan"))
    idx = torch.full((T, k), -1, dtype=torch.int32, device=dev)
    gate = torch.zeros((T, k), dtype=torch.float32, device=dev)
    pkg.moe_forward(shape, pkg.make_weights(w_t), x_t, y, idx, gate, ws)
    torch.cuda.synchronize()
    return y, idx.cpu().numpy(), gate.cpu().numpy().astype(np.float64)


def _forward_case(dev, oracle, cfg, T, w_np=None, w_t=None, sample=None, residual=False):
    """moe_forward vs the oracle.  sample: compare y only on that many seeded tokens (routing
    is always compared on all of them)."""
    if w_np is None:
        w_np = wl.make_layer_weights(cfg)
    if w_t is None:
        w_t = weights_to_device(w_np, dev)
    x_np = wl.make_inputs(cfg, T)
    y, idx, gate = _forward_gpu(dev, w_t, to_device(x_np, dev), cfg.top_k, DT[cfg.act_dtype], residual)
    same, _, _ = _check_routing(oracle, x_np, w_np, cfg.top_k, idx, gate)
    got = to_f64(y)
    assert np.all(np.isfinite(got))
    toks = np.arange(T)
    if sample is not None and sample < T:
        toks = np.sort(np.random.default_rng(cfg.seed).choice(T, size=sample, replace=False))
    toks = toks[same[toks]]
    ref, ridx, _ = oracle.forward(w_np, np.ascontiguousarray(x_np[toks]), cfg.top_k, residual=residual)
    assert np.array_equal(ridx, idx[toks])
    err = rel_err(got[toks], ref)
    tol = TOL[cfg.act_dtype]
    assert err < tol, f"{cfg.name} T={T}: relative error {err:.3e} >= {tol}"
    # no row may hide behind the norm of the whole tensor, and no sizeable element may be far off
    row_err = row_rel_err(got[toks], ref)
    assert row_err < tol, f"{cfg.name} T={T}: worst row's relative error {row_err:.3e} >= {tol}"
    elem_err = elementwise_rel_err(got[toks], ref)
    assert elem_err < ELEMENTWISE_TOL[cfg.act_dtype], \
        f"{cfg.name} T={T}: worst element-wise relative error {elem_err:.3e}"
    print(f"[parity] {cfg.name} T={T} tokens compared={len(toks)} tensor={err:.3e} worst-row={row_err:.3e} "
          f"worst-element={elem_err:.3e}")
    return err


def test_forward_tiny_fp32_config(dev, oracle):
    cfg = wl.CONFIGS["tiny"]
    _forward_case(dev, oracle, cfg, 32)
    _forward_case(dev, oracle, cfg, 1)
    _forward_case(dev, oracle, cfg, 5, residual=True)


@pytest.mark.parametrize("T", [1, 2, 3, 130, 512, 1024, 20000])
def test_forward_wearables_config(dev, oracle, T):
    # 130 and 512: 64-row GEMM tiles (and two k-groups for the down product); 1024: 128-row tiles;
    # 20000: 256-row tiles over many m-tiles and the multi-workgroup sort inside the forward
    _forward_case(dev, oracle, wl.CONFIGS["wearables"], T, sample=1024)  # all tokens but at T = 20000


@pytest.mark.parametrize("T", [1, 40, 700])
def test_forward_many_experts(dev, oracle, T):
    cfg = _cfg(name="e64", d=256, F=512, E=64, k=8, dtype="bf16", seed=640, std=0.05)
    _forward_case(dev, oracle, cfg, T)


@pytest.fixture(scope="module")
def phone(dev):
    cfg = wl.CONFIGS["phone"]
    w_np = wl.make_layer_weights(cfg)
    return cfg, w_np, weights_to_device(w_np, dev)


def test_forward_phone_config_decode_and_prefill(dev, oracle, phone):
    cfg, w_np, w_t = phone
    _forward_case(dev, oracle, cfg, 1, w_np, w_t)
    _forward_case(dev, oracle, cfg, 2048, w_np, w_t)  # every token's output is compared
    # the stored router bias must realise the Zipf(1.1) expert loads it was calibrated for
    x_np = wl.make_inputs(cfg, 2048)
    idx, _, _, _ = oracle.route(x_np, w_np["router_w"], w_np["router_b"], cfg.top_k)
    share = np.bincount(idx.reshape(-1), minlength=8) / idx.size
    assert np.abs(share - wl.zipf_target_shares(8, 1.1)).max() < 0.01


def test_staged_calls_at_the_phone_prefill_size(dev, oracle, phone):
    # route -> permute (with the gather) -> expert FFN -> combine through the four staged entry
    # points at the size the benchmark runs: the staged expert FFN takes the single-output down
    # projection (128 x 128 tiles), which moe_forward no longer does at this size
    cfg, w_np, w_t = phone
    T, k, E, d = 2048, cfg.top_k, cfg.n_experts, cfg.d_model
    x_np = wl.make_inputs(cfg, T)
    x_t = to_device(x_np, dev)
    shape = pkg.shape_for(w_t, T, k, pkg.MOE_BF16)
    P = T * k
    idx = torch.empty((T, k), dtype=torch.int32, device=dev)
    gate = torch.empty((T, k), dtype=torch.float32, device=dev)
    pkg.moe_route(shape, x_t, w_t["router_w"], w_t["router_b"], idx, gate, None)
    off = torch.empty(E + 1, dtype=torch.int32, device=dev)
    perm = torch.empty(P, dtype=torch.int32, device=dev)
    inv = torch.empty(P, dtype=torch.int32, device=dev)
    xp = torch.empty((P, d), dtype=torch.bfloat16, device=dev)
    pkg.moe_permute(shape, idx, off, perm, inv, x_t, xp, pkg.alloc_workspace(shape, dev))
    yp = torch.full_like(xp, float("nan"))
    ffn_shape = pkg.shape_for(w_t, P, 1, pkg.MOE_BF16)
    pkg.moe_expert_ffn(ffn_shape, pkg.make_weights(w_t), xp, off, yp, pkg.alloc_workspace(ffn_shape, dev))
    y = torch.full_like(x_t, float("nan"))
    pkg.moe_combine(shape, yp, inv, gate, None, y)
    torch.cuda.synchronize()
    idx_np = idx.cpu().numpy()
    same, _, _ = _check_routing(oracle, x_np, w_np, k, idx_np, gate.cpu().numpy().astype(np.float64))
    r_off, r_perm, r_inv = oracle.permute(idx_np, E)
    assert np.array_equal(off.cpu().numpy(), r_off) and np.array_equal(perm.cpu().numpy(), r_perm)
    assert np.array_equal(inv.cpu().numpy(), r_inv)
    toks = np.sort(np.random.default_rng(5).choice(T, size=512, replace=False))
    toks = toks[same[toks]]
    ref, _, _ = oracle.forward(w_np, np.ascontiguousarray(x_np[toks]), k)
    got = to_f64(y)
    assert np.all(np.isfinite(got))
    assert rel_err(got[toks], ref) < TOL["bf16"] and row_rel_err(got[toks], ref) < TOL["bf16"]
    # and against moe_forward on the same input (k-parts in its down projection: close, not equal)
    y_fwd, idx_fwd, _ = _forward_gpu(dev, w_t, x_t, k, pkg.MOE_BF16)
    assert np.array_equal(idx_fwd, idx_np)
    assert rel_err(to_f64(y_fwd), got) < 1e-2


@pytest.mark.parametrize("static", [False, True])
def test_forward_replayed_from_a_hip_graph_matches_eager(dev, static):
    # a prefill step and a single-token step captured into one graph and replayed several times with
    # eager work and synchronisations between the replays: every replay must reproduce the eager bits
    cfg = wl.shrink(wl.CONFIGS["wearables"], d_model=512, d_ff=1024)
    w_t = weights_to_device(wl.make_layer_weights(cfg), dev)
    k = cfg.top_k
    xs = [to_device(wl.make_inputs(cfg, T, step=T), dev) for T in (96, 1)]
    shapes = [pkg.shape_for(w_t, x.shape[0], k, pkg.MOE_BF16) for x in xs]
    wss = [pkg.alloc_workspace(sh, dev) for sh in shapes]
    weights = pkg.make_weights(w_t)

    def run(outs):
        for x, sh, ws, (y, idx, gate) in zip(xs, shapes, wss, outs):
            if static:
                pkg.moe_forward_static(sh, weights, x, y, idx, gate)
            else:
                pkg.moe_forward(sh, weights, x, y, idx, gate, ws)

    def fresh():
        return [(torch.full_like(x, float("nan")), torch.full((x.shape[0], k), -1, dtype=torch.int32, device=dev),
                 torch.zeros((x.shape[0], k), dtype=torch.float32, device=dev)) for x in xs]

    eager = fresh()
    run(eager)
    torch.cuda.synchronize()
    captured = fresh()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run(captured)  # warm-up on the capture stream (one-time set-up calls happen here, not under capture)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            run(captured)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    for rep in range(4):
        for y, idx, gate in captured:  # clear with fill kernels, outside the graph
            y.fill_(float("nan"))
            idx.fill_(-1)
        other = fresh()
        run(other)  # eager work between the replays, on the same scratch
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for (y, idx, gate), (ye, ie, ge), (yo, io, go) in zip(captured, eager, other):
            assert torch.equal(y, ye) and torch.equal(idx, ie) and torch.equal(gate, ge), f"replay {rep}"
            assert torch.equal(yo, ye)


@pytest.mark.parametrize("T", [2, 3, 5, 8])
def test_forward_phone_config_few_tokens(dev, oracle, phone, T):
    # a row or two per expert
    cfg, w_np, w_t = phone
    _forward_case(dev, oracle, cfg, T, w_np, w_t)
    _forward_case(dev, oracle, cfg, T, w_np, w_t, residual=True)


@pytest.mark.parametrize("d,F,E,k,r,base,T", [
    # one and two MFMA row blocks: 15, 16, 17, 31 and 32 rows in a group (k = E puts every token in each), the
    # first size past them; K of one piece of 16 bytes, a step and a bit, an odd number of steps per wave;
    # 8 of 16 columns in the last block; one part of K or more
    (40, 72, 3, 3, 0, False, 15), (264, 1160, 4, 4, 0, False, 16), (1032, 2056, 2, 2, 0, False, 17),
    (2040, 4104, 2, 2, 0, False, 31), (488, 8184, 2, 2, 0, False, 32), (488, 8200, 2, 2, 0, False, 3), (264, 520, 4, 4, 0, False, 33),
    (2048, 2824, 64, 1, 0, False, 3), (1440, 3840, 9, 7, 0, False, 2), (776, 2072, 64, 8, 0, False, 32), (776, 2072, 4, 2, 0, False, 2),
    (2056, 1064, 4, 2, 0, False, 9), (136, 1056, 5, 2, 0, False, 1 + 8),
    # rank factors (two activation operands), alone and beside a shared base
    (520, 1384, 4, 2, 264, False, 3), (1600, 4264, 8, 2, 800, False, 17), (1800, 1048, 3, 3, 1544, False, 19), (264, 3080, 2, 2, 8, False, 32),
    (520, 1384, 4, 2, 24, True, 2), (1000, 2728, 4, 3, 72, True, 20), (264, 1048, 4, 1, 40, True, 12),
])
def test_forward_few_rows_per_group(dev, oracle, d, F, E, k, r, base, T):
    cfg = _cfg(name="few", d=d, F=F, E=E, k=k, dtype="bf16", seed=1700 + d + F + T, r=r, base=base, std=0.03)
    _forward_case(dev, oracle, cfg, T, residual=bool(T % 2))


@pytest.mark.parametrize("d,F,r,offsets", [
    (72, 1000, 0, [0, 16, 16, 17]), (264, 520, 0, [0, 0, 31, 32]), (1032, 2056, 136, [0, 1, 20, 20, 27]), (2048, 96, 0, [0, 1]),
])
def test_expert_ffn_few_rows_per_group(dev, oracle, d, F, r, offsets):
    cfg = _cfg(d=d, F=F, E=len(offsets) - 1, dtype="bf16", seed=1750 + d + r, r=r, std=0.04)
    _ffn_case(dev, oracle, cfg, np.array(offsets, np.int32), TOL["bf16"])


@pytest.mark.parametrize("d,F,E,k,r,T", [
    # large weights in rows of 1, 2, 3, 4, 5 and 7 eighths of a line past whole ones, both widths and k-steps that
    # end before, at and after the shift of a row; one to four parts; groups of less than a tile, of one and of several
    (1032, 2760, 8, 2, 0, 40), (1056, 2784, 8, 2, 0, 129), (1240, 3224, 8, 2, 0, 257), (1000, 2728, 8, 2, 0, 384), (1016, 2808, 8, 1, 0, 700),
    (1400, 3736, 4, 2, 0, 257), (2040, 5624, 2, 1, 0, 384), (1992, 3160, 3, 3, 0, 129), (1040, 2776, 7, 2, 0, 384), (2040, 2728, 8, 2, 1160, 129),
    # gate and up alone, and the first sizes at which they are
    (904, 2440, 8, 2, 0, 129), (856, 2304, 8, 2, 0, 41), (840, 2336, 8, 2, 0, 300),
])
def test_forward_weights_in_cut_lines(dev, oracle, d, F, E, k, r, T):
    cfg = _cfg(name="cut", d=d, F=F, E=E, k=k, dtype="bf16", seed=1800 + d + T, r=r, std=0.03)
    _forward_case(dev, oracle, cfg, T, residual=bool(T % 2))


@pytest.mark.parametrize("d,F,offsets", [
    (1400, 3736, [0, 0, 128, 257, 300]), (1032, 2760, [0, 1, 2, 258, 258, 270, 398, 399, 400]), (2040, 5624, [0, 130, 131]),
])
def test_expert_ffn_weights_in_cut_lines(dev, oracle, d, F, offsets):
    cfg = _cfg(d=d, F=F, E=len(offsets) - 1, dtype="bf16", seed=1850 + d, r=0, std=0.03)
    _ffn_case(dev, oracle, cfg, np.array(offsets, np.int32), TOL["bf16"])


@pytest.mark.parametrize("d,F,E,k,T", [
    # a down projection in one part with few row tiles: 64 and 128 rows, widths below, at and past 128 columns and not multiples of
    # 16, K of 512 and a ragged one, and more tiles than a round
    (120, 512, 4, 2, 70), (128, 520, 4, 2, 130), (136, 1000, 8, 2, 300), (640, 1728, 8, 2, 512), (440, 1152, 3, 3, 400), (1024, 576, 8, 2, 1000),
    (1032, 576, 8, 2, 1000),
])
def test_forward_narrow_down_tiles(dev, oracle, d, F, E, k, T):
    cfg = _cfg(name="narrow", d=d, F=F, E=E, k=k, dtype="bf16", seed=1870 + d + T, r=0, std=0.04)
    _forward_case(dev, oracle, cfg, T, residual=bool(T % 4))


def _forward_guarded(w_t, x_t, k, act):
    """moe_forward on y, idx, gate and workspace that each lie between guard bytes, which have to be as they were."""
    T, shape = x_t.shape[0], pkg.shape_for(w_t, x_t.shape[0], k, act)
    sizes = [x_t.numel() * x_t.element_size(), T * k * 4, T * k * 4, pkg.moe_workspace_bytes(shape)]
    bufs = [torch.full((4096 + n + 4096,), 0xA5, dtype=torch.uint8, device=x_t.device) for n in sizes]
    y, idx, gate, ws = (b[4096:4096 + n] for b, n in zip(bufs, sizes))
    y, idx, gate = y.view(x_t.dtype).view(x_t.shape), idx.view(torch.int32).view(T, k), gate.view(torch.float32).view(T, k)
    idx.fill_(-1)
    pkg.moe_forward(shape, pkg.make_weights(w_t), x_t, y, idx, gate, ws)
    torch.cuda.synchronize()
    for b, n, what in zip(bufs, sizes, ("y", "idx", "gate", "workspace")):
        assert bool((b[:4096] == 0xA5).all()) and bool((b[4096 + n:] == 0xA5).all()), f"written outside {what}"
    return y, idx, gate


@pytest.mark.parametrize("same_experts", [False, True])
@pytest.mark.parametrize("T,k,E,dtype", [(32, 2, 5, "bf16"), (9, 3, 40, "bf16"), (17, 2, 5, "f32")])
def test_forward_few_tokens_some_with_nan_logits(dev, T, k, E, dtype, same_experts):
    # such a token's pairs may land in one expert or in none.  The others are, bit for bit, what they are beside finite tokens (a
    # row of a tile does not depend on where it lies or what the others hold), also where all tokens share their experts
    cfg = _cfg(name="nan", d=264, F=520, E=E, k=k, dtype=dtype, seed=1790 + E)
    w_t = weights_to_device(wl.make_layer_weights(cfg), dev)
    if same_experts:
        w_t["router_b"] = torch.zeros(E, dtype=torch.float32, device=dev)
        w_t["router_b"][E - k:] = 100.0
    x_t = to_device(wl.make_inputs(cfg, T), dev)
    clean = _forward_guarded(w_t, x_t, k, DT[dtype])
    assert bool(torch.isfinite(clean[0]).all()) and (not same_experts or bool((clean[1] >= E - k).all()))
    bad = torch.zeros(T, dtype=torch.bool, device=dev)
    bad[[0, T // 2, T - 1]] = True
    x_bad = x_t.clone()
    x_bad[bad] = float("nan")
    mixed = _forward_guarded(w_t, x_bad, k, DT[dtype])
    for got, want, what in zip(mixed, clean, ("y", "idx", "gate")):
        assert torch.equal(got[~bad], want[~bad]), what
    x_t.fill_(float("nan"))  # no finite token at all: the call ends, inside its memory
    _forward_guarded(w_t, x_t, k, DT[dtype])


@pytest.mark.parametrize("d,F,E,k,T", [
    # every token with every expert: 16-token blocks with 1, 2, 15, 16 and 17 tokens in the last, one expert and the most,
    # an odd number, widths below a block and a k-step, a ragged k-step, eight k-steps and more per row
    (128, 256, 4, 2, 2), (8, 8, 1, 1, 3), (24, 40, 3, 2, 15), (136, 264, 5, 5, 16), (128, 256, 4, 1, 17), (264, 184, 16, 4, 33),
    (512, 1400, 2, 1, 31), (1024, 1024, 3, 3, 18), (64, 136, 8, 2, 256), (72, 376, 8, 8, 130),
    # the first sizes past it: inner widths, model width, tokens
    (64, 3080, 1, 1, 9), (1032, 72, 2, 1, 5), (256, 640, 4, 1, 200), (128, 184, 17, 2, 20),
])
def test_forward_small_fp32_layer(dev, oracle, d, F, E, k, T):
    cfg = _cfg(name="small", d=d, F=F, E=E, k=k, dtype="f32", seed=1800 + d + F + T, std=0.05)
    _forward_case(dev, oracle, cfg, T, residual=bool(T % 2))


@pytest.mark.parametrize("d,F,E,k,T", [
    # k-steps of a wave of the two products: none and 1, 1 and 2, 2 and 3, 3 and 4, 4 and 5, 7 and 8 -- whole turns of 3 or 4 and what is left
    (56, 104, 4, 2, 3), (136, 264, 4, 1, 2), (136, 264, 4, 1, 19), (264, 488, 4, 2, 3), (392, 1000, 2, 2, 20), (520, 600, 2, 2, 2), (520, 600, 2, 1, 17),
    (968, 904, 3, 2, 4),
])
def test_forward_small_fp32_layer_k_steps_of_a_wave(dev, oracle, d, F, E, k, T):
    _forward_case(dev, oracle, _cfg(name="steps", d=d, F=F, E=E, k=k, dtype="f32", seed=1850 + d + T, std=0.05), T)


@pytest.mark.parametrize("T,k,E", [(20, 2, 5), (3, 4, 16)])
def test_forward_small_fp32_layer_with_infinite_experts(dev, T, k, E):
    # an expert that a token did not choose leaves no trace in it, whatever its weights
    cfg = _cfg(name="inf", d=128, F=72, E=E, k=k, dtype="f32", seed=1890 + E, std=0.05)
    w_t = weights_to_device(wl.make_layer_weights(cfg), dev)
    x_t = to_device(wl.make_inputs(cfg, T), dev)
    y0, idx, _ = _forward_gpu(dev, w_t, x_t, k, pkg.MOE_F32)
    e = int(idx[0, 0])
    w_t["w_gate"][e].fill_(float("nan"))
    w_t["w_down"][e].fill_(float("inf"))
    y1, idx1, _ = _forward_gpu(dev, w_t, x_t, k, pkg.MOE_F32)
    assert np.array_equal(idx, idx1)
    hit = torch.from_numpy((idx == e).any(axis=1))
    assert torch.equal(y0.cpu()[~hit], y1.cpu()[~hit]) and bool(torch.isnan(y1.cpu()[hit]).all())


@pytest.mark.parametrize("T", [2, 3, 16, 33])
def test_small_fp32_layer_is_as_close_to_64_bits_as_single_tokens(dev, T):
    # A token alone takes the matrix-vector path.  Both errors are those of 32-bit sums in different orders: the ratio of one layer scatters by
    # 10 %, of the geometric mean over these 24 by 2 %; a single chain of products over all k-steps is at 1.5
    ratios = []
    for d, F, E, k in [(64, 152, 4, 1), (72, 168, 4, 2), (128, 256, 4, 2), (136, 360, 8, 1), (208, 496, 4, 2), (248, 608, 2, 2), (480, 1288, 2, 2),
                       (504, 1264, 2, 1)]:
        for seed in range(3):
            w_t = weights_to_device(wl.make_layer_weights(_cfg(d=d, F=F, E=E, k=k, dtype="f32", seed=1900 + 10 * seed + d)), dev)
            x_t = to_device(wl.make_inputs(_cfg(d=d, F=F, E=E, k=k, dtype="f32", seed=2000 + 10 * seed + d), T), dev)
            y, idx, gate = _forward_gpu(dev, w_t, x_t, k, pkg.MOE_F32)
            one = torch.cat([_forward_gpu(dev, w_t, x_t[t:t + 1].clone(), k, pkg.MOE_F32)[0] for t in range(T)])
            w64 = {n: v.double() for n, v in w_t.items() if v is not None}
            ref = torch.zeros(T, d, dtype=torch.float64, device=dev)
            for t in range(T):
                x = x_t[t].double()
                logits = w64["router_w"] @ x + w64.get("router_b", 0.0)
                p = torch.softmax(logits[torch.from_numpy(idx[t]).long().to(dev)], 0)
                for j, e in enumerate(idx[t]):
                    z = w64["w_gate"][e] @ x
                    ref[t] += p[j] * (w64["w_down"][e] @ (z * torch.sigmoid(z) * (w64["w_up"][e] @ x)))
            err, err_one = ((v.double() - ref).norm() for v in (y, one))
            ratios.append(float(err / err_one))
    mean = float(np.exp(np.mean(np.log(ratios))))
    assert mean <= 1.15, (mean, ratios)


@pytest.mark.parametrize("name,T", [("phone_wd", 2), ("phone_wd", 7), ("phone_wd_base", 2)])
def test_forward_weight_decomposed_few_tokens(dev, oracle, name, T):
    # pure L R experts: four matrix-vector stages with per-token and per-pair inputs; a shared base
    # keeps the grouped GEMM at these sizes
    cfg = wl.CONFIGS[name]
    _forward_case(dev, oracle, cfg, T)


@pytest.mark.parametrize("k,E,T,dtype", [(32, 64, 2, "bf16"), (33, 64, 2, "bf16"), (3, 5, 2, "f32"), (1, 4, 2, "bf16"),
                                         (7, 9, 2, "bf16"), (8, 64, 3, "bf16")])
def test_forward_few_tokens_pair_limits(dev, oracle, k, E, T, dtype):
    # two tokens on the matrix-vector path: 64 pairs is the most it takes (2 x 33 go to the grouped
    # GEMM); odd k makes a group of two pairs span both tokens; k = 1 is one pair per token
    cfg = _cfg(name=f"ft{k}{E}", d=264, F=520, E=E, k=k, dtype=dtype, seed=1300 + k + E + T, std=0.05)
    _forward_case(dev, oracle, cfg, T, residual=bool(k % 2))


@pytest.mark.parametrize("name", ["phone_wd", "phone_wd_base"])
def test_forward_phone_weight_decomposed_configs(dev, oracle, name):
    cfg = wl.CONFIGS[name]
    w_np = wl.make_layer_weights(cfg)
    w_t = weights_to_device(w_np, dev)
    _forward_case(dev, oracle, cfg, 1, w_np, w_t)
    _forward_case(dev, oracle, cfg, 2048, w_np, w_t)  # every token's output is compared


def test_forward_small_shapes_all_expert_kinds(dev, oracle):
    for dtype in ("f32", "bf16"):
        for r, base in ((0, False), (64, False), (24, True)):
            cfg = _cfg(name=f"s{r}{base}", d=192, F=328, E=5, k=3, dtype=dtype, seed=500 + r,
                       r=r, base=base, std=0.05)
            for T in (1, 7, 150):
                _forward_case(dev, oracle, cfg, T, residual=(T == 7))


def _sweep_cases(n, seed):
    """n seeded (d, F, E, k, r, base, dtype, T) combinations: widths any multiple of 8, from
    narrower than one k-step of the GEMM to a few tiles wide; token counts from one to a few
    hundred; every expert kind."""
    rng = np.random.default_rng(seed)
    cases = []
    for _ in range(n):
        d = 8 * int(rng.integers(1, 41))
        F = 8 * int(rng.integers(1, 65))
        E = int(rng.integers(1, 13))
        k = int(rng.integers(1, E + 1))
        kind = int(rng.integers(0, 3))  # dense / pure L R / shared base + L R
        r = 0 if kind == 0 else 8 * int(rng.integers(1, 9))
        dtype = "f32" if rng.integers(0, 4) == 0 else "bf16"
        T = int(rng.choice([1, 2, 3, 5, 17, 64, 129, 300, 400]))
        cases.append((d, F, E, k, r, kind == 2, dtype, T))
    return cases


@pytest.mark.parametrize("d,F,E,k,r,base,dtype,T", _sweep_cases(28, 20250300245))
def test_forward_seeded_shape_sweep(dev, oracle, d, F, E, k, r, base, dtype, T):
    cfg = _cfg(name="sw", d=d, F=F, E=E, k=k, dtype=dtype, seed=7000 + d + F + E + k + r + T, r=r,
               base=base, std=0.08)
    _forward_case(dev, oracle, cfg, T, residual=bool((d + T) % 2))


def _prefill_sweep_cases(n, seed):
    """n seeded prefill-sized combinations: a few hundred rows per expert and widths up to a dozen
    tiles, so the 256- and 128-row GEMM kernels run with K tails, ragged groups and cut tiles."""
    rng = np.random.default_rng(seed)
    cases = []
    for _ in range(n):
        d = 8 * int(rng.integers(16, 160))
        F = 8 * int(rng.integers(32, 400))
        E = int(rng.integers(2, 9))
        k = int(rng.integers(1, min(E, 4) + 1))
        kind = int(rng.integers(0, 3))
        r = 0 if kind == 0 else 8 * int(rng.integers(2, 33))
        T = int(rng.integers(600, 3000))
        cases.append((d, F, E, k, r, kind == 2, T))
    return cases


@pytest.mark.parametrize("d,F,E,k,r,base,T", _prefill_sweep_cases(10, 2503))
def test_forward_seeded_prefill_sweep(dev, oracle, d, F, E, k, r, base, T):
    cfg = _cfg(name="pf", d=d, F=F, E=E, k=k, dtype="bf16", seed=8000 + d + F + E + k + r + T, r=r,
               base=base, std=0.04)
    _forward_case(dev, oracle, cfg, T, sample=256)


@pytest.mark.parametrize("d,F,E,k,T", [
    (256, 2048, 3, 2, 1500),   # 32 steps of 64 cut into 4 parts of 8
    (256, 2080, 2, 1, 2000),   # 32 whole steps and a tail of 32: only the last part holds the tail
    (512, 4128, 2, 2, 1100),   # 64.5 steps, two output tiles per row tile
    (1792, 2048, 8, 2, 96), (1792, 2048, 8, 2, 97),   # parts in fp32 up to 24 rows per expert, in bf16 from there on
])
def test_forward_down_projection_cut_along_k(dev, oracle, d, F, E, k, T):
    # tall groups, a narrow output and a long K: the down projection's 256 x 256 tiles are too few
    # for the chip, so moe_forward cuts every tile's k-steps into parts whose partial outputs the
    # combine adds; the result must still match the oracle and the staged calls (one part) closely
    cfg = _cfg(name="kp", d=d, F=F, E=E, k=k, dtype="bf16", seed=1200 + F, std=0.04)
    w_np = wl.make_layer_weights(cfg, with_bias=False)
    w_t = weights_to_device(w_np, dev)
    _forward_case(dev, oracle, cfg, T, w_np, w_t, sample=300)
    # staged calls on the same input
    x_t = to_device(wl.make_inputs(cfg, T), dev)
    y1, idx1, _ = _forward_gpu(dev, w_t, x_t, k, pkg.MOE_BF16)
    shape = pkg.shape_for(w_t, T, k, pkg.MOE_BF16)
    P = T * k
    idx = torch.empty((T, k), dtype=torch.int32, device=dev)
    gate = torch.empty((T, k), dtype=torch.float32, device=dev)
    pkg.moe_route(shape, x_t, w_t["router_w"], None, idx, gate, None)
    off = torch.empty(E + 1, dtype=torch.int32, device=dev)
    perm = torch.empty(P, dtype=torch.int32, device=dev)
    inv = torch.empty(P, dtype=torch.int32, device=dev)
    xp = torch.empty((P, d), dtype=torch.bfloat16, device=dev)
    pkg.moe_permute(shape, idx, off, perm, inv, x_t, xp, pkg.alloc_workspace(shape, dev))
    yp = torch.empty_like(xp)
    ffn_shape = pkg.shape_for(w_t, P, 1, pkg.MOE_BF16)
    pkg.moe_expert_ffn(ffn_shape, pkg.make_weights(w_t), xp, off, yp, pkg.alloc_workspace(ffn_shape, dev))
    y3 = torch.empty_like(x_t)
    pkg.moe_combine(shape, yp, inv, gate, None, y3)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), idx1)
    assert rel_err(to_f64(y1), to_f64(y3)) < 1e-2  # bf16 parts are rounded one by one


@pytest.mark.parametrize("d,F,T", [(256, 2048, 3), (256, 2048, 90), (512, 4096, 16), (256, 1152, 500), (512, 4096, 700)])
def test_forward_down_projection_whose_halves_of_k_cancel(dev, oracle, d, F, T):
    # Hidden unit j + F/2 repeats unit j, and its column of the down projection is minus that of j but for a
    # 128th: the halves of K are about a hundred times their sum.  One fp32 sum, or fp32 parts of it, is off by
    # some 100 x 2^-24 x sqrt(F), far below the rounding of the result; parts rounded to bf16 (2^-9 each) would
    # be off by half of it.
    cfg = _cfg(name="cancel", d=d, F=F, E=4, k=2, dtype="bf16", seed=1300 + F + T, std=0.04)
    w_np = wl.make_layer_weights(cfg, with_bias=False)
    for name in ("w_gate", "w_up"):
        w_np[name][:, F // 2:] = w_np[name][:, :F // 2]
    w_np["w_down"][:, :, F // 2:] = wl.f32_to_bf16_bits(
        wl.bf16_bits_to_f32(w_np["w_down"][:, :, :F // 2]) * np.float32(-127 / 128))
    _forward_case(dev, oracle, cfg, T, w_np, sample=100)


@pytest.mark.parametrize("k,E,T", [(2, 8, 2), (2, 8, 37), (2, 8, 600), (3, 5, 150), (8, 8, 64), (2, 16, 9)])
def test_forward_shared_base_once_per_token(dev, oracle, k, E, T):
    # bf16 layers with k > 1 take the path that applies the shared base once per token (plain
    # products over T rows, low-rank terms per pair, the shared down term added in the combine);
    # T = 9 with 16 experts leaves most groups empty, T = 600 spans several tiles
    cfg = _cfg(name=f"tb{k}{E}", d=256, F=448, E=E, k=k, dtype="bf16", seed=900 + k + E, r=64,
               base=True, std=0.05)
    _forward_case(dev, oracle, cfg, T, residual=(T == 37))


@pytest.mark.parametrize("T", [5, 300, 1500])
def test_forward_shared_base_once_per_token_ragged_widths(dev, oracle, T):
    # the same path with widths that are multiples of 8 only: every product has a K tail
    # (200 = 3 x 64 + 8, 328 = 5 x 64 + 8, rank 40 is shorter than one k-step)
    cfg = _cfg(name="tbr", d=200, F=328, E=4, k=2, dtype="bf16", seed=931, r=40, base=True, std=0.05)
    _forward_case(dev, oracle, cfg, T)


@pytest.mark.parametrize("d,F,E,k,r,base,dtype", [
    # row lengths of one vector, one chunk less / more a vector, four chunks and one vector more (its own router launch)
    (8, 8, 2, 1, 0, False, "bf16"), (504, 520, 4, 2, 0, False, "bf16"), (1032, 1544, 8, 4, 0, False, "bf16"),
    (2048, 6144, 8, 2, 0, False, "bf16"), (2056, 6152, 8, 2, 0, False, "bf16"), (328, 8200, 16, 16, 0, False, "bf16"),
    (264, 1000, 5, 3, 0, False, "bf16"), (64, 128, 64, 8, 0, False, "bf16"),
    (8, 16, 2, 2, 0, False, "f32"), (264, 2056, 8, 4, 0, False, "f32"), (1024, 1032, 4, 1, 0, False, "f32"),
    (1032, 264, 8, 2, 0, False, "f32"),
    (200, 328, 8, 2, 104, False, "bf16"), (520, 1064, 4, 1, 264, False, "bf16"),          # rank factors
    (8, 8, 3, 3, 8, False, "bf16"), (2048, 5632, 8, 2, 1024, False, "bf16"), (264, 8200, 8, 3, 520, False, "bf16"),
    (328, 1064, 8, 4, 1544, False, "bf16"), (392, 72, 16, 7, 256, False, "bf16"), (72, 4104, 4, 2, 1536, False, "bf16"),
    (8, 8, 2, 2, 8, True, "bf16"), (264, 520, 8, 3, 24, True, "bf16"), (1544, 4104, 16, 4, 136, True, "bf16"),  # shared base
    (520, 512, 8, 2, 520, True, "bf16"),                                                  # d above F: the general kernels
    (2048, 5632, 8, 2, 64, True, "bf16"),
])
@pytest.mark.parametrize("residual", [False, True])
def test_forward_one_token(dev, oracle, d, F, E, k, r, base, dtype, residual):
    cfg = _cfg(d=d, F=F, E=E, k=k, dtype=dtype, seed=520 + d + k, r=r, base=base, std=0.05)
    _forward_case(dev, oracle, cfg, 1, residual=residual)


@pytest.mark.parametrize("d,F,E,k,r,base,dtype", [
    # more (pair, row) units than waves (4096): a rest of 8, of three quarters and 8 more, none; rows of no whole lines, then of whole lines
    (72, 8200, 4, 1, 0, False, "bf16"), (72, 5640, 4, 2, 0, False, "bf16"), (72, 5632, 4, 2, 0, False, "bf16"), (72, 4096, 4, 2, 0, False, "bf16"),
    (64, 4104, 4, 1, 0, False, "bf16"), (64, 5640, 4, 2, 0, False, "bf16"), (64, 5632, 4, 2, 0, False, "bf16"), (40, 4104, 4, 3, 0, False, "f32"),
    (72, 4104, 4, 2, 16, True, "bf16"), (128, 8000, 4, 2, 16, True, "bf16"),  # a shared base's rows, on the other workgroups
])
def test_forward_one_token_rest_of_the_rows(dev, oracle, d, F, E, k, r, base, dtype):
    cfg = _cfg(name="rest", d=d, F=F, E=E, k=k, r=r, base=base, dtype=dtype, seed=977 + d, std=0.05)
    _forward_case(dev, oracle, cfg, 1)


@pytest.mark.parametrize("F,k,r", [
    # rows of a pair's rank factors on 4096 / k waves: one turn, a row past it, a last turn of three quarters and 8 rows more, two whole turns
    (2048, 2, 264), (2056, 2, 520), (3584, 2, 264), (3592, 2, 264), (4096, 2, 1032), (2384, 3, 264), (2392, 3, 264), (4104, 1, 520), (1800, 4, 264),
    (2056, 2, 320), (4096, 2, 320), (3592, 2, 320), (1800, 4, 512),  # rows of whole lines
    (1192, 6, 264), (504, 14, 264),  # (as many rows as workgroups have waves for: the last one lacks one of some pairs)
])
def test_forward_one_token_rank_experts_last_turn_of_rows(dev, oracle, F, k, r):
    _forward_case(dev, oracle, _cfg(name="turn", d=72, F=F, E=max(4, k), k=k, r=r, dtype="bf16", seed=1210 + F, std=0.05), 1)


@pytest.mark.parametrize("d,F,E,k,r", [
    # blocks of 64 hidden rows whole and not, one block, ranks of one vector and whole ones, the most pairs and the most sums; the first
    # sizes past it: a longer rank, more sums
    (64, 64, 4, 4, 8), (200, 1096, 8, 2, 64), (1032, 4104, 16, 4, 64), (328, 8200, 32, 32, 8), (136, 200, 8, 8, 32), (1000, 2680, 8, 2, 24),
    (200, 456, 4, 4, 72), (264, 520, 8, 5, 56),
])
def test_forward_one_token_shared_base_rank_down_in_parts(dev, oracle, d, F, E, k, r):
    cfg = _cfg(d=d, F=F, E=E, k=k, dtype="bf16", seed=540 + d + k, r=r, base=True, std=0.05)
    w_np = wl.make_layer_weights(cfg)
    w_t = weights_to_device(w_np, dev)
    for residual in (False, True):
        _forward_case(dev, oracle, cfg, 1, w_np=w_np, w_t=w_t, residual=residual)
    _forward_guarded(w_t, to_device(wl.make_inputs(cfg, 1), dev), k, pkg.MOE_BF16)


@pytest.mark.parametrize("r,base", [(0, False), (264, False), (64, True), (72, True)])  # (a base's ranks: in parts, and past them)
@pytest.mark.parametrize("E", [5, 40])
def test_forward_one_token_with_nan_logits(dev, E, r, base):
    # no order among NaN logits: whichever lanes a round names, the weights read are an expert's, and nothing is written beside the outputs
    cfg = _cfg(d=264, F=520, E=E, dtype="bf16", seed=560 + E, r=r, base=base, std=0.05)
    w_t = weights_to_device(wl.make_layer_weights(cfg), dev)
    x_t = to_device(wl.make_inputs(cfg, 1), dev)
    y, _, _ = _forward_guarded(w_t, torch.full_like(x_t, float("nan")), cfg.top_k, DT["bf16"])
    assert torch.isnan(y).all()
    assert np.all(np.isfinite(to_f64(_forward_gpu(dev, w_t, x_t, cfg.top_k, DT["bf16"])[0])))


@pytest.mark.parametrize("E,k,T,dtype", [
    (1, 1, 1, "f32"), (5, 3, 341, "f32"), (64, 8, 129, "f32"), (8, 2, 2048, "f32"), (8, 1, 4097, "f32"),  # up to 4096 pairs
    (3, 1, 5, "bf16"), (8, 2, 1024, "bf16"), (64, 8, 257, "bf16"), (7, 3, 1001, "bf16"),                  # up to 8192
    (8, 2, 4096, "bf16"), (8, 1, 8193, "bf16"),
])
def test_forward_sorts_the_pairs_in_its_first_product(dev, E, k, T, dtype):
    # the sorted order that moe_forward uses inside equals moe_permute's: same products on the same rows
    cfg = _cfg(d=128, F=136, E=E, k=k, dtype=dtype, seed=700 + T, std=0.05)
    w_t = weights_to_device(wl.make_layer_weights(cfg), dev)
    x_t = to_device(wl.make_inputs(cfg, T), dev)
    y, idx, gate = _forward_gpu(dev, w_t, x_t, k, DT[dtype])
    shape, P = pkg.shape_for(w_t, T, k, DT[dtype]), T * k
    off = torch.empty(E + 1, dtype=torch.int32, device=dev)
    perm, inv = (torch.empty(P, dtype=torch.int32, device=dev) for _ in range(2))
    xp = torch.empty((P, cfg.d_model), dtype=x_t.dtype, device=dev)
    pkg.moe_permute(shape, torch.from_numpy(idx).to(dev), off, perm, inv, x_t, xp, pkg.alloc_workspace(shape, dev))
    ffn_shape, yp, y2 = pkg.shape_for(w_t, P, 1, DT[dtype]), torch.empty_like(xp), torch.empty_like(x_t)
    pkg.moe_expert_ffn(ffn_shape, pkg.make_weights(w_t), xp, off, yp, pkg.alloc_workspace(ffn_shape, dev))
    pkg.moe_combine(shape, yp, inv, torch.from_numpy(gate.astype(np.float32)).to(dev), None, y2)
    torch.cuda.synchronize()
    assert rel_err(to_f64(y), to_f64(y2)) < (1e-6 if dtype == "f32" else 1e-3)


@pytest.mark.parametrize("E,k,T", [
    # both ways of counting and both sides of their lines (2048 pairs, 8 experts), pairs that are no multiple of 4, every thread full
    (8, 1, 2047), (8, 1, 2049), (8, 2, 1025), (9, 1, 2051), (9, 3, 683), (5, 1, 6143), (2, 1, 8191), (8, 4, 2048), (64, 2, 4093),
])
@pytest.mark.parametrize("skew", [False, True])
def test_forward_counts_the_pairs_of_an_expert(dev, E, k, T, skew):
    # all experts are one and the same but for the output columns that they write, which no two share: a pair in a wrong group leaves its own columns zero,
    # and a row of another token is off by its whole size, whatever the pair's gate
    d = 64
    cfg = _cfg(d=d, F=64, E=E, k=k, dtype="bf16", seed=730 + T, std=0.05)
    w_t = weights_to_device(wl.make_layer_weights(cfg), dev)
    if skew:
        w_t["router_b"] = torch.linspace(2.0, 0.0, E, dtype=torch.float32, device=dev)
    for name in ("w_gate", "w_up", "w_down"):
        w_t[name] = w_t[name][:1].expand_as(w_t[name]).contiguous()
    owner = torch.arange(d, device=dev) // (d // E)  # of a column (E and beyond: nobody's)
    w_t["w_down"] *= (owner == torch.arange(E, device=dev)[:, None])[:, :, None]
    x_t = to_device(wl.make_inputs(cfg, T), dev)
    w = {n: w_t[n].double() for n in ("w_gate", "w_up", "w_down")}
    y, idx, gate = _forward_gpu(dev, w_t, x_t, k, pkg.MOE_BF16)
    x, down = x_t.double(), w["w_down"].sum(0)
    z = x @ w["w_gate"][0].T
    one = ((z * torch.sigmoid(z)) * (x @ w["w_up"][0].T)) @ down.T
    gates = torch.zeros(T, E + 1, dtype=torch.float64, device=dev)
    gates.scatter_(1, torch.from_numpy(idx).long().to(dev), torch.from_numpy(gate).double().to(dev))
    g = gates[:, owner.clamp(max=E)]
    got = torch.from_numpy(to_f64(y)).to(dev)
    assert bool((got[g == 0] == 0).all())
    # h, the pairs' outputs and y are rounded to bf16, 2^-9 of a value each: against the root mean square of what an expert writes for the token, of which a value is
    # five and a half at the most here, 0.03
    size = one.square().mean(1, keepdim=True).sqrt() * g
    assert float(((got - one * g).abs() / size)[g != 0].max()) < 0.05


def test_forward_is_deterministic_and_matches_the_staged_calls(dev, oracle):
    cfg = wl.shrink(wl.CONFIGS["wearables"], d_model=512, d_ff=1024)
    w_np = wl.make_layer_weights(cfg)
    w_t = weights_to_device(w_np, dev)
    T, k = 200, cfg.top_k
    x_t = to_device(wl.make_inputs(cfg, T), dev)
    y1, idx1, gate1 = _forward_gpu(dev, w_t, x_t, k, pkg.MOE_BF16)
    y2, idx2, gate2 = _forward_gpu(dev, w_t, x_t, k, pkg.MOE_BF16)
    assert torch.equal(y1, y2) and np.array_equal(idx1, idx2) and np.array_equal(gate1, gate2)
    # staged pipeline through the same ABI
    shape = pkg.shape_for(w_t, T, k, pkg.MOE_BF16)
    ws = pkg.alloc_workspace(shape, dev)
    P = T * k
    idx = torch.empty((T, k), dtype=torch.int32, device=dev)
    gate = torch.empty((T, k), dtype=torch.float32, device=dev)
    pkg.moe_route(shape, x_t, w_t["router_w"], None, idx, gate, None)
    off = torch.empty(cfg.n_experts + 1, dtype=torch.int32, device=dev)
    perm = torch.empty(P, dtype=torch.int32, device=dev)
    inv = torch.empty(P, dtype=torch.int32, device=dev)
    xp = torch.empty((P, cfg.d_model), dtype=torch.bfloat16, device=dev)
    pkg.moe_permute(shape, idx, off, perm, inv, x_t, xp, ws)
    yp = torch.empty_like(xp)
    ffn_shape = pkg.shape_for(w_t, P, 1, pkg.MOE_BF16)
    pkg.moe_expert_ffn(ffn_shape, pkg.make_weights(w_t), xp, off, yp, pkg.alloc_workspace(ffn_shape, dev))
    y3 = torch.empty_like(x_t)
    pkg.moe_combine(shape, yp, inv, gate, None, y3)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), idx1)          # routing bit-identical
    assert np.array_equal(gate.cpu().numpy().astype(np.float64), gate1)
    assert torch.equal(y3, y1)                               # same kernels, same bits


# ------------------------------------------------------------------------------- moe_stack_forward

def _stack_case(dev, oracle, cfg, n_layers, T):
    layers_np = wl.make_stack_weights(cfg, n_layers)
    layers_t = [weights_to_device(w, dev) for w in layers_np]
    x_np = wl.make_inputs(cfg, T)
    act = DT[cfg.act_dtype]
    shape = pkg.shape_for(layers_t[0], T, cfg.top_k, act)
    ws = pkg.alloc_workspace(shape, dev)
    x_t = to_device(x_np, dev)
    y = torch.empty_like(x_t)
    trace = torch.full((n_layers, T, cfg.top_k), -1, dtype=torch.int32, device=dev)
    pkg.moe_stack_forward(shape, [pkg.make_weights(w) for w in layers_t], x_t, y, trace, ws)
    torch.cuda.synchronize()
    y_ref, trace_ref, xs = oracle.stack_forward(layers_np, x_np, cfg.top_k)
    trace = trace.cpu().numpy()
    # free-running: compare the final residual on tokens whose routing never flipped
    clean = np.all(trace == trace_ref, axis=(0, 2))
    assert clean.mean() > 0.9, "too many routing flips for near-tie noise"
    err = rel_err(to_f64(y)[clean], y_ref[clean])
    assert err < TOL[cfg.act_dtype], f"stack error {err:.3e}"
    # teacher-forced: each GPU layer fed the oracle's (storage-rounded) input of that layer
    for l in range(n_layers):
        xin = xs[l].astype(np.float32)
        xin = xin if cfg.act_dtype == "f32" else wl.f32_to_bf16_bits(xin)
        yl, idx, gate = _forward_gpu(dev, layers_t[l], to_device(xin, dev), cfg.top_k, act, residual=True)
        same, _, _ = _check_routing(oracle, xin, layers_np[l], cfg.top_k, idx, gate)
        ref, _, _ = oracle.forward(layers_np[l], xin, cfg.top_k, residual=True)
        assert rel_err(to_f64(yl)[same], ref[same]) < TOL[cfg.act_dtype]


def test_stack_small(dev, oracle):
    cfg = wl.shrink(wl.CONFIGS["phone_stack"], d_model=256, d_ff=512, weight_std=0.05)
    _stack_case(dev, oracle, cfg, 5, 1)
    _stack_case(dev, oracle, cfg, 4, 40)


def test_stack_phone_width_decode(dev, oracle):
    _stack_case(dev, oracle, wl.CONFIGS["phone_stack"], 3, 1)


def test_stack_phone_full_depth_decode_loop(dev, oracle):
    """The fifth benchmark configuration at its stated size: 24 phone-shaped layers with
    residual adds, one token per step, several steps with a fresh N(0,1) token each.
    Teacher-forced, every layer of every step: the GPU layer is fed the oracle's input of that
    layer (rounded to bf16); routing must be bit-exact off the ambiguous set and the output
    within tolerance.  Free-running, to the end of the stack: the final residual stream is
    compared on the steps whose routing never left the oracle's; flips are counted and printed."""
    cfg = wl.CONFIGS["phone_stack"]
    n_layers, n_steps, k = cfg.n_layers, 6, cfg.top_k
    assert n_layers == 24
    layers_np = wl.make_stack_weights(cfg, n_layers)
    layers_t = [weights_to_device(w, dev) for w in layers_np]
    structs = [pkg.make_weights(w) for w in layers_t]
    shape = pkg.shape_for(layers_t[0], 1, k, pkg.MOE_BF16)
    ws = pkg.alloc_workspace(shape, dev)
    clean_steps, free_errs, forced_worst, n_amb = 0, [], 0.0, 0
    for step in range(n_steps):
        x_np = wl.make_inputs(cfg, 1, step=step)
        x_t = to_device(x_np, dev)
        y = torch.full_like(x_t, float("nan"))
        trace = torch.full((n_layers, 1, k), -1, dtype=torch.int32, device=dev)
        pkg.moe_stack_forward(shape, structs, x_t, y, trace, ws)
        torch.cuda.synchronize()
        y_ref, trace_ref, xs = oracle.stack_forward(layers_np, x_np, k)
        tr = trace.cpu().numpy()
        flips = int(np.any(tr != trace_ref, axis=(1, 2)).sum())
        first_flip = int(np.argmax(np.any(tr != trace_ref, axis=(1, 2)))) if flips else -1
        got = to_f64(y)
        assert np.all(np.isfinite(got))
        err = rel_err(got, y_ref)
        growth = float(np.sqrt(np.mean(y_ref ** 2)))
        print(f"[stack24] step {step}: layers whose routing differs {flips} (first at {first_flip}), "
              f"free-running error of the final stream {err:.3e}, rms of the final stream {growth:.2f}")
        if flips == 0:
            clean_steps += 1
            free_errs.append(err)
            assert err < TOL["bf16"], f"step {step}: free-running error {err:.3e} at depth {n_layers}"
        # teacher-forced, layer by layer
        for l in range(n_layers):
            xin = wl.f32_to_bf16_bits(xs[l].astype(np.float32))
            yl, idx, gate = _forward_gpu(dev, layers_t[l], to_device(xin, dev), k, pkg.MOE_BF16, residual=True)
            same, _, _ = _check_routing(oracle, xin, layers_np[l], k, idx, gate)
            n_amb += int((~same).sum())
            if same[0]:
                ref, _, _ = oracle.forward(layers_np[l], xin, k, residual=True)
                e = rel_err(to_f64(yl), ref)
                assert e < TOL["bf16"], f"step {step} layer {l}: teacher-forced error {e:.3e}"
                # the stream is mostly the residual, so also compare the layer's own contribution
                yc, idx_c, _ = _forward_gpu(dev, layers_t[l], to_device(xin, dev), k, pkg.MOE_BF16)
                assert np.array_equal(idx_c, idx)
                ref_c, _, _ = oracle.forward(layers_np[l], xin, k)
                ec = rel_err(to_f64(yc), ref_c)
                assert ec < TOL["bf16"], f"step {step} layer {l}: error of the layer's contribution {ec:.3e}"
                forced_worst = max(forced_worst, e, ec)
    print(f"[stack24] {clean_steps}/{n_steps} steps without a routing flip, worst free-running error on them "
          f"{max(free_errs) if free_errs else float('nan'):.3e}; worst teacher-forced layer error {forced_worst:.3e}; "
          f"teacher-forced ambiguous picks {n_amb}")
    assert clean_steps >= 1, "every step's routing left the oracle's somewhere in the 24 layers"


# ------------------------------------------------------------------------------- routing-trace metrics

def _fig5_trace(name):
    import os
    m = np.loadtxt(os.path.join(os.path.dirname(__file__), "golden", name), dtype=np.int64, comments="#")
    return np.stack([np.flatnonzero(m[:, t]) for t in range(m.shape[1])]).astype(np.int32)[None]


def _random_trace(seed, B, T, K, E, sticky=0.7):
    """Selections that change only now and then, like a router with temporal locality."""
    rng = np.random.default_rng(seed)
    S = np.zeros((B, T, K), np.int32)
    for b in range(B):
        cur = rng.permutation(E)[:K]
        for t in range(T):
            if rng.random() > sticky:
                cur = cur.copy()
                cur[rng.integers(K)] = rng.choice(np.setdiff1d(np.arange(E), cur)) if E > K else cur[0]
            S[b, t] = rng.permutation(cur)
    return S


@pytest.mark.parametrize("case", ["fig5_bles", "fig5_moe", "random", "single_token", "wide", "long"])
def test_expert_replacements_match_oracle_bit_exact(dev, oracle, case):
    if case.startswith("fig5"):
        S, E = _fig5_trace(case + ".txt"), 8
    elif case == "random":
        S, E = _random_trace(1, 5, 333, 2, 8), 8
    elif case == "single_token":
        S, E = _random_trace(2, 4, 1, 2, 8), 8
    elif case == "wide":
        S, E = _random_trace(3, 2, 700, 8, 64, sticky=0.3), 64
    else:
        S, E = _random_trace(4, 24, 4096, 2, 8), 8
    He = torch.full((E,), -1, dtype=torch.int64, device=dev)
    H = torch.full((1,), -1, dtype=torch.int64, device=dev)
    pkg.moe_expert_replacements(to_device(S, dev), E, He, H)
    torch.cuda.synchronize()
    rH, rHe = oracle.expert_replacements(S, E)
    assert int(H.item()) == rH and np.array_equal(He.cpu().numpy(), rHe)
    if case == "fig5_bles":
        assert rH // 2 == 11
    if case == "fig5_moe":
        assert rH // 2 == 21


@pytest.mark.parametrize("B,T,K,E", [(1, 2, 1, 2), (3, 257, 2, 8), (2, 2048, 2, 8), (1, 1, 2, 4), (4, 100, 8, 64)])
def test_bles_loss_value_matches_oracle(dev, oracle, B, T, K, E):
    rng = np.random.default_rng(B * 1000 + T)
    W = rng.random((B, T, E)).astype(np.float32) ** 3
    W /= W.sum(-1, keepdims=True)
    S = np.argsort(-W, axis=-1, kind="stable")[..., :K].astype(np.int32)
    out = torch.full((5,), float("nan"), dtype=torch.float64, device=dev)
    ws = torch.empty(pkg.moe_bles_workspace_bytes(B, T, E), dtype=torch.uint8, device=dev)
    pkg.moe_bles_loss(to_device(W, dev), to_device(S, dev), out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    ref = oracle.bles_loss(W, S)
    assert got[0] == ref["H"] and got[1] == ref["H_norm"]          # integer part exact
    for i, key in ((2, "L"), (3, "L_norm"), (4, "loss")):            # fp32 block sums, fp64 total
        assert abs(got[i] - ref[key]) <= 2e-6 * max(abs(ref[key]), 1e-30), (key, got[i], ref[key])


@pytest.mark.parametrize("B,T,K,E", [
    # traces of one workgroup: the shortest, turns that are not full, sequences shorter and longer than a turn, one expert a
    # token, ballots and atomics, the longest by pairs and by elements and the first sizes past them, many layers
    # the limits of each call, by tokens, experts, chunks of a row, layers and pairs of a layer, and the first sizes past them
    (1, 4096, 1, 8), (1, 4097, 1, 6), (1, 3072, 2, 8), (3, 1025, 2, 8), (8, 384, 2, 9), (7, 439, 2, 9), (1, 384, 1, 64), (1, 2048, 1, 3),
    (8, 512, 2, 8), (17, 180, 2, 8), (17, 181, 2, 8), (32, 96, 4, 8), (33, 2, 2, 8), (16, 128, 8, 16), (15, 137, 8, 16), (1, 256, 8, 16), (1, 257, 8, 16),
])
def test_trace_statistics_of_short_traces(dev, oracle, B, T, K, E):
    S = _random_trace(B + T, B, T, K, E)
    W = np.random.default_rng(B + T).random((B, T, E), np.float32)
    He, H = torch.full((E,), -1, dtype=torch.int64, device=dev), torch.full((1,), -1, dtype=torch.int64, device=dev)
    counts = torch.full((B, E), -1, dtype=torch.int64, device=dev)
    delta, mean = torch.full((B,), -1.0, dtype=torch.float64, device=dev), torch.full((1,), -1.0, dtype=torch.float64, device=dev)
    out = torch.full((5,), -1.0, dtype=torch.float64, device=dev)
    ws = torch.empty(pkg.moe_bles_workspace_bytes(B, T, E), dtype=torch.uint8, device=dev)
    S_gpu = to_device(S, dev)
    pkg.moe_expert_replacements(S_gpu, E, He, H)
    pkg.moe_bles_loss(to_device(W, dev), S_gpu, out, ws)
    pkg.moe_delta_uniform(S_gpu, E, counts, delta, mean)
    torch.cuda.synchronize()
    rH, rHe = oracle.expert_replacements(S, E)
    assert int(H.item()) == rH and np.array_equal(He.cpu().numpy(), rHe)
    # differences and the sum of four in fp32 (up to 6 roundings of 2^-24 each), the rest in fp64
    ref = np.abs(np.diff(W.astype(np.float64), axis=1)).sum() if T > 1 else 0.0
    got = out.cpu().numpy()
    assert got[0] == rH and abs(got[2] - ref) <= 6 * 2.0 ** -24 * ref and got[4] == got[1] * got[3]
    r_mean, r_delta, r_counts = oracle.delta_uniform(S, E)
    assert np.array_equal(counts.cpu().numpy(), r_counts)
    assert np.allclose(delta.cpu().numpy(), r_delta, rtol=1e-14, atol=1e-16)
    assert abs(mean.item() - r_mean) <= 1e-13 * max(r_mean, 1e-30) + 1e-16


@pytest.mark.parametrize("B,T,E,offset", [(1, 2048, 64, 0), (3, 700, 8, 0), (2, 999, 7, 0), (1, 4096, 64, 1), (9000, 2, 8, 0)])
def test_bles_loss_adds_its_differences_in_fp64(dev, B, T, E, offset):
    # Probabilities that alternate between 0 and c: every difference is c, and so is exact, as are the sums of
    # the four of one 16-byte load.  What is left are fp64 sums; fp32 ones of more terms would round in one
    # direction (1e-8 and more of the result).  B T tokens in pairs (T = 2) need more partial sums per element
    # than the workspace holds for long sequences.  offset: rows that are not 16-byte aligned.
    c = np.float32(1 / 3)
    store = torch.zeros(B * T * E + offset, dtype=torch.float32, device=dev)
    W = store[offset:].view(B, T, E)
    W[:, 1::2] = float(c)
    S = torch.zeros((B, T, 1), dtype=torch.int32, device=dev)
    S[:, 1::2] = 1
    out = torch.full((5,), -1.0, dtype=torch.float64, device=dev)
    ws = torch.empty(pkg.moe_bles_workspace_bytes(B, T, E) + 4, dtype=torch.uint8, device=dev)
    for ws_at in (0, 4):
        out.fill_(-1.0)
        pkg.moe_bles_loss(W, S, out, ws[ws_at:])
        torch.cuda.synchronize()
        H, Hn, L, Ln, loss = out.cpu().tolist()
        ref = float(c) * B * (T - 1) * E
        assert H == 2 * B * (T - 1) and Hn == 1.0
        assert abs(L - ref) <= 1e-13 * ref and abs(Ln - ref / (B * T)) <= 1e-13 * ref / (B * T)
        assert loss == Ln


def test_bles_loss_from_the_routers_own_probabilities(dev, oracle):
    cfg = _cfg(d=256, E=8, k=2, dtype="bf16", seed=77, std=0.3)
    w_np = wl.make_layer_weights(cfg, with_bias=False)
    B, T = 3, 200
    x_np = wl.make_inputs(cfg, B * T)
    w_t = weights_to_device({"router_w": w_np["router_w"], "router_b": None}, dev)
    idx, gate, probs = _route_gpu(dev, to_device(x_np, dev), w_t, 8, 2, pkg.MOE_BF16)
    probs_t = to_device(probs.astype(np.float32).reshape(B, T, 8), dev)
    S_t = to_device(idx.reshape(B, T, 2), dev)
    out = torch.zeros(5, dtype=torch.float64, device=dev)
    ws = torch.empty(pkg.moe_bles_workspace_bytes(B, T, 8), dtype=torch.uint8, device=dev)
    pkg.moe_bles_loss(probs_t, S_t, out, ws)
    torch.cuda.synchronize()
    ref = oracle.bles_loss(probs.astype(np.float32).reshape(B, T, 8), idx.reshape(B, T, 2))
    got = out.cpu().numpy()
    assert got[0] == ref["H"] and abs(got[4] - ref["loss"]) <= 2e-6 * ref["loss"]
    assert 0.0 < ref["loss"] < 2.0


@pytest.mark.parametrize("L,T,K,E", [(1, 35, 2, 8), (24, 256, 2, 8), (3, 1, 2, 4), (2, 1000, 4, 16), (5, 300, 8, 64)])
def test_offload_counters_match_oracle_bit_exact(dev, oracle, L, T, K, E):
    tr = _fig5_trace("fig5_moe.txt") if (L, T) == (1, 35) else _random_trace(L + T, L, T, K, E, sticky=0.6)
    ch = torch.full((L,), -1, dtype=torch.int64, device=dev)
    ld = torch.full((L,), -1, dtype=torch.int64, device=dev)
    pkg.moe_offload_counters(to_device(tr, dev), E, ch, ld)
    torch.cuda.synchronize()
    rch, rld = oracle.offload_counters(tr, E)
    assert np.array_equal(ch.cpu().numpy(), rch) and np.array_equal(ld.cpu().numpy(), rld)
    if (L, T) == (1, 35):
        assert rld[0] == 2 + 21  # the paper's 21 replacements after the initial fill


@pytest.mark.parametrize("case", ["fig5", "random", "single_token", "wide", "long", "collapsed", "stray"])
def test_delta_uniform_matches_oracle(dev, oracle, case):
    if case == "fig5":
        tr, E = _fig5_trace("fig5_moe.txt"), 8
    elif case == "random":
        tr, E = _random_trace(21, 5, 333, 2, 8), 8
    elif case == "single_token":
        tr, E = _random_trace(22, 4, 1, 2, 8), 8
    elif case == "wide":
        tr, E = _random_trace(23, 3, 700, 8, 64, sticky=0.3), 64
    elif case == "long":
        tr, E = _random_trace(24, 3, 70000, 2, 8), 8   # several chunks per layer
    elif case == "collapsed":
        tr, E = np.tile(np.array([[6, 1]], np.int32), (2, 50, 1)), 8
    else:
        tr, E = _random_trace(25, 2, 90, 2, 8), 8
    L = tr.shape[0]
    counts = torch.full((L, E), -1, dtype=torch.int64, device=dev)
    delta = torch.full((L,), float("nan"), dtype=torch.float64, device=dev)
    mean = torch.full((1,), float("nan"), dtype=torch.float64, device=dev)
    tr_gpu = tr.copy()
    if case == "stray":
        tr_gpu[1, 7, 0] = -3   # entries outside [0, E) are ignored by the library (the oracle rejects them)
        tr_gpu[0, 3, 1] = E
    pkg.moe_delta_uniform(to_device(tr_gpu, dev), E, counts, delta, mean)
    torch.cuda.synchronize()
    r_mean, r_delta, r_counts = oracle.delta_uniform(tr, E)
    if case == "stray":
        r_counts[1, tr[1, 7, 0]] -= 1
        r_counts[0, tr[0, 3, 1]] -= 1
        assert np.array_equal(counts.cpu().numpy(), r_counts)
        return
    assert np.array_equal(counts.cpu().numpy(), r_counts)            # integer part bit-exact
    # fp64 on both sides, the same operations in the same order
    assert np.allclose(delta.cpu().numpy(), r_delta, rtol=1e-14, atol=1e-16)
    assert abs(mean.item() - r_mean) <= 1e-14 * max(r_mean, 1e-30) + 1e-16
    if case == "collapsed":
        assert mean.item() == 1.5


def test_stack_trace_feeds_the_trace_metrics(dev, oracle):
    cfg = wl.shrink(wl.CONFIGS["phone_stack"], d_model=256, d_ff=512, weight_std=0.05)
    n_layers, T = 6, 64
    layers_np = wl.make_stack_weights(cfg, n_layers)
    layers_t = [weights_to_device(w, dev) for w in layers_np]
    shape = pkg.shape_for(layers_t[0], T, cfg.top_k, pkg.MOE_BF16)
    ws = pkg.alloc_workspace(shape, dev)
    x_t = to_device(wl.make_inputs(cfg, T), dev)
    y = torch.empty_like(x_t)
    trace = torch.empty((n_layers, T, cfg.top_k), dtype=torch.int32, device=dev)
    pkg.moe_stack_forward(shape, [pkg.make_weights(w) for w in layers_t], x_t, y, trace, ws)
    ch = torch.empty(n_layers, dtype=torch.int64, device=dev)
    ld = torch.empty(n_layers, dtype=torch.int64, device=dev)
    He = torch.empty(cfg.n_experts, dtype=torch.int64, device=dev)
    H = torch.empty(1, dtype=torch.int64, device=dev)
    pkg.moe_offload_counters(trace, cfg.n_experts, ch, ld)
    pkg.moe_expert_replacements(trace, cfg.n_experts, He, H)
    torch.cuda.synchronize()
    tr = trace.cpu().numpy()
    rch, rld = oracle.offload_counters(tr, cfg.n_experts)
    rH, rHe = oracle.expert_replacements(tr, cfg.n_experts)
    assert np.array_equal(ch.cpu().numpy(), rch) and np.array_equal(ld.cpu().numpy(), rld)
    assert int(H.item()) == rH and np.array_equal(He.cpu().numpy(), rHe)
    # loads after the initial fill of k experts per layer are exactly the replacements
    assert int(rld.sum()) - n_layers * cfg.top_k == rH // 2


# ------------------------------------------------------------------------------- the paper's own shapes

@pytest.mark.parametrize("d,F,r", [
    (1440, 3840, 0),     # phone-sized MoE row of Table 1 (hidden 1440, F = 8h/3)
    (432, 1152, 0),      # wearable-sized MoE row (hidden 432)
    (1600, 4264, 800),   # phone-sized WD row: hidden 1600, rank = hidden / 2
    (400, 1064, 200),    # wearable-sized WD row
])
def test_forward_table1_shapes(dev, oracle, d, F, r):
    # widths that are not multiples of the GEMM's K tile exercise its K tail
    cfg = _cfg(name=f"t1_{d}", d=d, F=F, E=8, k=2, dtype="bf16", seed=600 + d, r=r, std=0.03)
    w_np = wl.make_layer_weights(cfg, with_bias=False)
    w_t = weights_to_device(w_np, dev)
    _forward_case(dev, oracle, cfg, 1, w_np, w_t)
    _forward_case(dev, oracle, cfg, 150, w_np, w_t)
    # a prefill batch: 512 rows per expert on average, the 256-row tiles with their K tails
    _forward_case(dev, oracle, cfg, 2048, w_np, w_t, sample=512)


@pytest.mark.parametrize("E", [2, 4, 8, 16])
@pytest.mark.parametrize("k", [1, 2, 4, 8])
def test_forward_active_and_total_expert_grid(dev, oracle, k, E):
    # the ablation grid of Sec. 3.5 (k active of 8 total; 2 active of E total), at a small width
    if k > E:
        pytest.skip("k cannot exceed E")
    cfg = _cfg(name=f"g{k}_{E}", d=256, F=384, E=E, k=k, dtype="bf16", seed=700 + 10 * k + E, std=0.05)
    w_np = wl.make_layer_weights(cfg, with_bias=False)
    w_t = weights_to_device(w_np, dev)
    _forward_case(dev, oracle, cfg, 1, w_np, w_t)
    _forward_case(dev, oracle, cfg, 70, w_np, w_t)
