"""The fused attention's decode routes, operand ranges, fold and schedule at
the sizes where they change, against the float64 oracle (Sec. 3.3).

Routes: a BFP8 page is decoded to BF16 on packed 16-bit integers where all its
block exponents lie in 7..133, else through float32; both are exact.  Operands:
softmax weights and queries keep BF16's exponent range, whatever lies beside
them.  Fold: the last workgroup of a (sequence, KV head) takes the partials in
batches of 8, 3, 2 and 1.  Schedule: in short ranges whole pieces go to single
waves.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import LSE_ATOL, LSE_RTOL, DevKV, assert_attn_close, bf16_bits_to_f64, note
from oracle_fixtures import PagedKV, make_paged, tiny_workload

pytestmark = pytest.mark.gpu

BF16_STEP = 2.0 ** -133          # the smallest BF16 magnitude


def _assert_close_by_row(out, lse, ref, ref_lse, what):
    """|gpu - ref| <= 2e-3 M + 1e-2 |ref| with M the largest |ref| of the same
    sequence and query head: the tolerance of every attention test at the
    values' own scale.  Its absolute part covers sums that cancel: some hundred
    terms of at most M / L each with 2^-17 relative error.  Where M itself is a
    BF16 subnormal the output's step adds two of them."""
    got = bf16_bits_to_f64(out)
    assert np.isfinite(got).all(), what
    top = np.abs(ref).max(axis=-1, keepdims=True)
    bound = 2e-3 * top + 1e-2 * np.abs(ref) + np.where(top < 2.0 ** -118, 2 * BF16_STEP, 0.0)
    err = np.abs(got - ref)
    assert (err <= bound).all(), f"{what}: {(err > bound).sum()} of {err.size}, worst {(err / bound).max():.3g} x bound"
    # an output of zeros, or off by a factor of two, would not pass
    assert ((np.abs(ref) / 2 > bound).any(axis=-1) | (top[..., 0] == 0)).all(), what
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, rtol=LSE_RTOL, atol=LSE_ATOL, err_msg=what)


def _exponents(kv, case, rng):
    """Per-page block exponents of K and V for a case, and the exponent of |q|
    that keeps the scores of order one; the pages' mantissas stay."""
    shape = kv.k_mant.shape[:3] + (kv.k_exp.shape[3],)
    if case == "usual":
        return rng.integers(120, 134, shape), rng.choice([120, 121, 132, 133], shape), -3
    if case == "packed_edges":               # both ends of the packed route, and one past each
        return rng.choice([123, 126, 7, 6], shape), rng.choice([6, 7, 133, 134], shape), 4
    if case == "one_past_in_a_page":         # one block of every third page leaves the packed route
        k, v = np.full(shape, 127), np.full(shape, 127)
        k[::3, :, 5, 2] = 134
        v[1::3, :, 9, 7] = 5
        return k, v, 0
    if case == "small":
        return np.full(shape, 101), rng.integers(84, 95, shape), 26
    if case == "large":
        return np.full(shape, 122), rng.integers(188, 199, shape), 4
    if case == "by_page":
        k, v = np.full(shape, 127), np.full(shape, 127)
        k[::3], v[::3] = 112, 99
        return k, v, 0
    if case == "subnormal_values":           # the smallest block exponents: BF16 subnormals
        return np.full(shape, 124), np.full(shape, 2), 3
    if case == "tiny_and_huge_values":       # V near 2^-40 in every second page, near 2^115 in the others
        v = np.full(shape, 87)
        v[1::2] = 242
        return np.full(shape, 124), v, 3
    raise ValueError(case)


def _decoded(kv):
    kv.k_bf16 = oracle.decode_blocks(kv.k_mant, kv.k_exp)
    kv.v_bf16 = oracle.decode_blocks(kv.v_mant, kv.v_exp)
    return kv


@pytest.mark.parametrize("group", [1, 8, 9])
@pytest.mark.parametrize("case", ["usual", "packed_edges", "one_past_in_a_page", "small", "large", "by_page",
                                  "subnormal_values", "tiny_and_huge_values"])
def test_routes_by_block_exponent(case, group):
    rng = np.random.default_rng(9000 + group)
    w = tiny_workload(Hq=2 * group, Hkv=2, B=4, index=50)
    note(f"attn routes: {case}, group {group}")
    kv = make_paged(w, ctx=[16, 33, 160, 527], garbage_tail=False)
    k, v, q_exp = _exponents(kv, case, rng)
    kv.k_exp[...], kv.v_exp[...] = k, v
    _decoded(kv)
    kv.q[:] = (kv.q & 0x807F) | np.uint16((127 + q_exp) << 7)      # 2^q_exp <= |q| < 2^(q_exp + 1)
    ref, ref_lse = kv.oracle_attn()
    # the scores matter: without them lse would be log(length)
    assert np.abs(ref_lse - np.log(kv.ctx)[:, None]).max() > 0.05
    for bf16_pages in (False, True):         # pure and mixed-format kernel
        for tps in (0, 64):
            out, lse = DevKV(kv).attn(tokens_per_split=tps, use_bf16_pools=bf16_pages)
            _assert_close_by_row(out, lse, ref, ref_lse, f"{case}, mixed {bf16_pages}, tps {tps}")


def _one_token_dominates(group, bits, ctx):
    """Every sequence's second token (or its only one) outweighs each of the others by 2^bits
    and has V = 0: the output is the others' values, times 2^-bits."""
    w = tiny_workload(Hq=2 * group, Hkv=2, B=len(ctx), index=53)
    kv = make_paged(w, ctx=ctx, garbage_tail=False)
    kv.k_mant[...], kv.k_exp[...], kv.v_exp[...] = 0, 127, 127
    kv.q[...] = 0
    kv.q[..., 0] = 0x4100                                      # 8
    want = bits * np.log(2.0) / (8 * kv.scale)                 # the dominating token's key, below 64
    for b in range(len(ctx)):
        page = kv.page_table[b, 0]
        kv.k_mant[page, :, 1, 0] = int(round(want * 2))        # times 2^(132 - 133)
        kv.k_exp[page, :, 1, 0] = 132
        kv.v_mant[page, :, 1] = 0
    return _decoded(kv)


@pytest.mark.parametrize("group", [1, 8, 16])
@pytest.mark.parametrize("bits", [20, 28, 36, 60])
def test_small_weights_beside_a_token_without_value(bits, group):
    note(f"attn: weights 2^-{bits}, group {group}")
    kv = _one_token_dominates(group, bits, [16, 19, 333])
    ref, ref_lse = kv.oracle_attn()
    for bf16_pages in (False, True):
        out, lse = DevKV(kv).attn(use_bf16_pools=bf16_pages)
        _assert_close_by_row(out, lse, ref, ref_lse, f"weights 2^-{bits}, mixed {bf16_pages}")


@pytest.mark.parametrize("group", [1, 8, 16])
def test_small_queries_beside_a_large_one(group):
    """A query channel of 2^40 that meets zeros in K leaves the others' scores as they are."""
    w = tiny_workload(Hq=2 * group, Hkv=2, B=3, index=54)
    note(f"attn: query of 2^40, group {group}")
    kv = make_paged(w, ctx=[16, 50, 333], garbage_tail=False)
    kv.k_mant[..., 37] = 0
    kv.q[..., 37] = (127 + 40) << 7
    _decoded(kv)
    ref, ref_lse = kv.oracle_attn()
    assert np.abs(ref_lse - np.log(kv.ctx)[:, None]).max() > 0.05
    for bf16_pages in (False, True):
        out, lse = DevKV(kv).attn(use_bf16_pools=bf16_pages)
        _assert_close_by_row(out, lse, ref, ref_lse, f"query of 2^40, mixed {bf16_pages}")


@pytest.mark.parametrize("bf16_pages", [False, True])
@pytest.mark.parametrize("values", ["encoded", "one_dominates"])
def test_bits_do_not_depend_on_slots_past_the_context(values, bf16_pages):
    """The same tokens with other bytes behind them: exponents inside and
    outside the packed route, infinities."""
    note(f"attn: tails, {values}, mixed {bf16_pages}")
    ctx = [1, 5, 15, 17, 333]
    if values == "encoded":
        kv = make_paged(tiny_workload(Hq=16, Hkv=2, B=len(ctx), index=55), ctx=ctx, garbage_tail=False)
    else:
        kv = _one_token_dominates(8, 40, ctx)
    got = []
    for tail in (None, 127, 134, 3, 255):
        if tail is not None:
            for b, n in enumerate(ctx):
                page, used = kv.page_table[b, (n - 1) // 16], (n - 1) % 16 + 1
                for mant, ex in ((kv.k_mant, kv.k_exp), (kv.v_mant, kv.v_exp)):
                    mant[page, :, used:] = 0xFF
                    ex[page, :, used:] = tail
        for tps in (0, 64):
            got.append((tps,) + DevKV(_decoded(kv)).attn(tokens_per_split=tps, use_bf16_pools=bf16_pages))
    for tps, out, lse in got[2:]:
        first = got[0 if tps == 0 else 1]
        assert torch.equal(out, first[1]) and torch.equal(lse, first[2])


@pytest.mark.parametrize("seed", range(4))
def test_formats_agree_bitwise_over_many_outputs(seed):
    """BFP8 pages and BF16 pages of the same values, under one schedule: half a
    million outputs a seed, every bit."""
    note(f"attn: formats, seed {seed}")
    rng = np.random.default_rng(9200 + seed)
    B, hq, hkv, pages = 64, 64, 8, 20
    n = B * pages
    mant = [rng.integers(0, 256, (n, hkv, 16, 128), dtype=np.uint8) for _ in range(2)]
    ex = [rng.integers(lo, hi, (n, hkv, 16, 8), dtype=np.uint8) for lo, hi in ((118, 124), (121, 133))]
    q = np.random.default_rng(seed).standard_normal((B, hq, 128)).astype(np.float32)
    q = (q.view(np.uint32) >> 16).astype(np.uint16)
    table = rng.permutation(n).astype(np.int32).reshape(B, pages)
    ctx = rng.integers(16 * pages - 15, 16 * pages + 1, B).astype(np.int32)
    kv = _decoded(PagedKV(q, mant[0], ex[0], mant[1], ex[1], None, None, table, ctx, hkv, 16, 128 ** -0.5))
    out, lse = DevKV(kv).attn(tokens_per_split=160, use_bf16_pools=False)
    kv.page_table = table | oracle.TAG_BF16
    out2, lse2 = DevKV(kv).attn(tokens_per_split=160)
    assert torch.equal(out, out2) and torch.equal(lse, lse2)


@pytest.mark.parametrize("parts", [1, 2, 3, 4, 5, 7, 8, 9, 11, 16, 19])
def test_fold_of_any_number_of_partials(parts):
    w = tiny_workload(Hq=16, Hkv=2, B=2, index=51)
    note(f"attn: fold of {parts} partials")
    kv = make_paged(w, ctx=[16 * parts, 16 * parts - 5])
    ref, ref_lse = kv.oracle_attn()
    d = DevKV(kv)
    out, lse = d.attn(tokens_per_split=16)
    assert_attn_close(out, lse, ref, ref_lse, what=f"{parts} partials")


@pytest.mark.parametrize("bf16_fraction", [0.0, 0.5])
@pytest.mark.parametrize("lengths", ["short", "long_and_short", "with_empty", "one_page", "two_in_a_range"])
def test_pieces_taken_by_single_waves(lengths, bf16_fraction):
    """More workgroups than CUs, ranges short enough that their pieces go to
    the waves in turn (of two BFP8 pieces: stay with the workgroup): whole sequences, cut ones (published by a wave, folded
    with pieces of whole workgroups), empty ones between them, and the order of
    arrival without effect (a repeat gives the same bits)."""
    rng = np.random.default_rng(9100)
    B, hkv = 150, 4
    ctx = {"short": rng.integers(1, 200, B), "long_and_short": rng.integers(1, 150, B),
           "with_empty": rng.integers(0, 90, B), "one_page": np.full(B, 16),
           "two_in_a_range": np.full(B, 128) - (np.arange(B) % 7 == 0)}[lengths].astype(np.int32)
    if lengths == "long_and_short":
        ctx[rng.choice(B, 30, replace=False)] = rng.integers(1200, 1700, 30)
    if lengths == "with_empty":
        ctx[rng.random(B) < 0.4] = 0
    w = tiny_workload(Hq=4 * hkv, Hkv=hkv, B=B, index=52)
    note(f"attn: pieces by wave, {lengths}, BF16 share {bf16_fraction}")
    kv = make_paged(w, ctx=ctx, bf16_fraction=bf16_fraction)
    ref, ref_lse = kv.oracle_attn()
    d = DevKV(kv)
    out, lse = d.attn()
    assert_attn_close(out, lse, ref, ref_lse, what=f"pieces by wave, {lengths}")
    again, lse2 = d.attn()
    assert (out == again).all() and (lse == lse2).all()
