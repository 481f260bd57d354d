"""Edges of the tiles, panels and splits that the kernels cut their work into, against the fp64 oracle.

The bounds are harness.check's: the parity bound of the types and, with fp32 records, the regression guard.
"""
import numpy as np
import pytest
import torch

import harness as H
from harness import oracle
from paper_2605_19049_amd import synth
from test_gpu_parity import _direct_case, _tree_case, _verify_case, say

pytestmark = pytest.mark.gpu

TYPES = [("bf16", "f32"), ("f16", "f32"), ("bf16", "bf16"), ("f16", "f16")]


@pytest.mark.parametrize("in_dtype, rec_dtype", TYPES)
@pytest.mark.parametrize("block_size", [None, 16])
def test_direct_second_panel(in_dtype, rec_dtype, block_size):
    """Contexts around the end of the first 64-row panel and around every 16-row block of the second."""
    lens = np.array([0, 1, 63, 64, 65, 66, 79, 80, 81, 95, 97, 112, 113, 127, 128], np.int32)
    e = _direct_case(B=len(lens), Hk=2, Hv=4, d=128, Lmax=128, cap=128, in_dtype=in_dtype, seed=800, lens=lens,
                     then_decode=False, rec_dtype=rec_dtype, out_dtype=rec_dtype, block_size=block_size)
    say("direct, second panel, %s/%s: rel err out/u/decode/state %.2e %.2e %.2e %.2e" % ((in_dtype, rec_dtype) + e))
    H.check(e, in_dtype, rec_dtype, "second panel")


@pytest.mark.parametrize("B, Hk, Hv", [(3, 8, 24), (5, 3, 9), (1, 1, 4), (2, 4, 4), (7, 16, 32), (13, 4, 8), (129, 2, 8)])
@pytest.mark.parametrize("Lmax", [33, 90])
def test_direct_every_unit_is_taken_once(B, Hk, Hv, Lmax):
    """Head counts that deal over the 8 XCDs and ones that do not; an untaken unit leaves NaN in its outputs."""
    e = _direct_case(B=B, Hk=Hk, Hv=Hv, d=128, Lmax=Lmax, cap=Lmax, in_dtype="bf16", seed=810 + B + Lmax)
    say("direct, B=%d heads %d/%d Lmax=%d: rel err out/u/decode/state %.2e %.2e %.2e %.2e" % ((B, Hk, Hv, Lmax) + e))
    H.check(e, "bf16", what="dealt units")


@pytest.mark.parametrize("d, in_dtype, rec_dtype", [(d, i, r) for d in (32, 64) for i, r in TYPES + [("f32", "f32")]]
                         + [(128, "f32", "f32")])
def test_direct_block_rows(d, in_dtype, rec_dtype):
    """The block-row kernel around every block of 16 rows, contiguous and paged (its bound is the 1e-5 of fp32
    workloads wherever records and outputs are fp32: accurate exponentials and exact products)."""
    lens = np.array([0, 1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64], np.int32)
    for block_size in (None, 8):
        e = _direct_case(B=len(lens), Hk=2, Hv=4, d=d, Lmax=64, cap=64, in_dtype=in_dtype, seed=820 + d, lens=lens,
                         then_decode=False, rec_dtype=rec_dtype, out_dtype=rec_dtype, block_size=block_size)
        say("direct, block rows, d=%d %s/%s: rel err out/u/decode/state %.2e %.2e %.2e %.2e" % ((d, in_dtype, rec_dtype) + e))
        H.check(e, "f32" if rec_dtype == "f32" else in_dtype, rec_dtype, "block rows")


@pytest.mark.parametrize("in_dtype, rec_dtype", TYPES)
@pytest.mark.parametrize("C", [1, 2, 15, 16, 17, 31, 32, 33, 48, 64, 65, 128])
def test_fused_update_tiles(in_dtype, rec_dtype, C):
    """The state update inside kvb_decode_flush around every 16-record tile and register window.  With fp32
    records the state is 1e7 times its usual size, so the delta values leave the range of fp16: the errors are
    relative, so the bounds stay what they are."""
    rng = np.random.default_rng(830 + C)
    S0 = H.prefix_state(rng, 2, 2, 4, 128, 128, in_dtype, 16)
    if rec_dtype == "f32":
        S0 = S0 * np.float32(1e7)
    tok = synth.token_stream(rng, 2, C + 3, 2, 4, 128, 128, in_dtype)
    lay = H.Layer(2, 2, 4, 128, 128, cap=C, in_dtype=in_dtype, scale=128 ** -0.5, rec_dtype=rec_dtype)
    o, u, S, _ = H.run_decode(lay, S0, tok, C, final_flush=False, fused=True)
    o_ref, u_ref, _ = oracle.kvb_decode_expected(S0, tok["q"], tok["k"], tok["v"], tok["g"], tok["beta"], scale=128 ** -0.5)
    # (the state holds what was folded: the first floor((C + 3) / C) * C tokens)
    n = (C + 3) // C * C
    _, _, S_ref = oracle.kvb_decode_expected(S0, *(tok[x][:, :n] for x in ("q", "k", "v", "g", "beta")), scale=128 ** -0.5)
    e = (H.rel_err(o, o_ref), H.rel_err(u, u_ref), H.rel_err(S, S_ref))
    say("fused update, %s/%s C=%d: rel err out/u/state %.2e %.2e %.2e" % ((in_dtype, rec_dtype, C) + e))
    H.check(e, in_dtype, rec_dtype, "fused update")


@pytest.mark.parametrize("C", [4, 5, 64, 65])
@pytest.mark.parametrize("d, in_dtype, rec_dtype", [(128, "bf16", "f32"), (128, "f16", "f16"), (64, "f32", "f32"), (32, "bf16", "f32")])
def test_fused_results_kept_or_sent_through(d, in_dtype, rec_dtype, C):
    """kvb_decode_flush on both sides of the thresholds from and up to which results stay in the cache: each step reads the
    records and, after two folds, the state that the steps before it left, in a buffer longer than the threshold."""
    rng = np.random.default_rng(970 + C)
    S0 = H.prefix_state(rng, 20, 2, 6, d, d, in_dtype, 16)
    tok = synth.token_stream(rng, 20, 2 * C + 2, 2, 6, d, d, in_dtype)
    lay = H.Layer(20, 2, 6, d, d, cap=max(16, C + 7), in_dtype=in_dtype, scale=d ** -0.5, rec_dtype=rec_dtype)
    o, u, S, _ = H.run_decode(lay, S0, tok, C, final_flush=False, fused=True)
    o_ref, u_ref, _ = oracle.kvb_decode_expected(S0, tok["q"], tok["k"], tok["v"], tok["g"], tok["beta"], scale=d ** -0.5)
    _, _, S_ref = oracle.kvb_decode_expected(S0, *(tok[x][:, :2 * C] for x in ("q", "k", "v", "g", "beta")), scale=d ** -0.5)
    e = (H.rel_err(o, o_ref), H.rel_err(u, u_ref), H.rel_err(S, S_ref))
    say("results kept or sent through, d=%d %s/%s C=%d: rel err out/u/state %.2e %.2e %.2e" % ((d, in_dtype, rec_dtype, C) + e))
    H.check(e, in_dtype, rec_dtype, "results kept or sent through")


@pytest.mark.parametrize("d, in_dtype, rec_dtype", [(128, "f32", "f32"), (64, "f32", "f32"), (64, "bf16", "f32"), (32, "f16", "f16")])
@pytest.mark.parametrize("C, block_size", [(9, None), (95, None), (128, 8)])
def test_flush_rows_chunks(d, in_dtype, rec_dtype, C, block_size):
    """kvb_flush off the 16-bit matrix instruction: remainders of a chunk of records, and several chunks."""
    rng = np.random.default_rng(840 + C)
    S0 = H.prefix_state(rng, 2, 2, 4, d, d, in_dtype, 16)
    tok = synth.token_stream(rng, 2, C + 3, 2, 4, d, d, in_dtype)
    lay = H.Layer(2, 2, 4, d, d, cap=C, in_dtype=in_dtype, scale=d ** -0.5, rec_dtype=rec_dtype, block_size=block_size)
    o, u, S, _ = H.run_decode(lay, S0, tok, C, fused=False)
    o_ref, u_ref, S_ref = oracle.kvb_decode_expected(S0, tok["q"], tok["k"], tok["v"], tok["g"], tok["beta"], scale=d ** -0.5)
    e = (H.rel_err(o, o_ref), H.rel_err(u, u_ref), H.rel_err(S, S_ref))
    say("flush rows, d=%d %s/%s C=%d: rel err out/u/state %.2e %.2e %.2e" % ((d, in_dtype, rec_dtype, C) + e))
    H.check(e, in_dtype, rec_dtype, "flush rows")


@pytest.mark.parametrize("d, in_dtype, rec_dtype", [(d, i, r) for d in (32, 64) for i, r in TYPES + [("f32", "f32")]]
                         + [(128, "f32", "f32")])
@pytest.mark.parametrize("C, T", [(1, 2), (16, 4), (30, 8), (60, 3), (120, 8)])
def test_verify_windows(d, in_dtype, rec_dtype, C, T):
    """kvb_verify and kvb_verify_tree off the 16-bit d = 128 path, in every record window and beyond it."""
    for block_size, case in ((None, _verify_case), (8, _tree_case)):
        cap = -(-(C - 1 + T) // 8) * 8
        e = case(5, 2, 6, d, C, cap, T, in_dtype, seed=850 + C, block_size=block_size, rec_dtype=rec_dtype)
        say("verify windows, d=%d %s/%s C=%d T=%d: %s" % (d, in_dtype, rec_dtype, C, T, e))
        H.check(e, in_dtype, rec_dtype, "verify windows")


@pytest.mark.parametrize("B, Hk, Hv, d, in_dtype, rec_dtype", [(45, 4, 12, 128, "f16", "f16"), (45, 4, 12, 128, "bf16", "f32"), (33, 4, 16, 64, "f32", "f32"),
                                                                (130, 4, 4, 32, "bf16", "bf16"), (20, 1, 2, 128, "f16", "f32"), (20, 2, 10, 32, "f32", "f32")])
@pytest.mark.parametrize("block_size", [None, 8])
def test_decode_from_the_buffer_alone(B, Hk, Hv, d, in_dtype, rec_dtype, block_size):
    """One and two heads to a workgroup, head ratios that two does not divide, fills around each block of records."""
    Lmax, cap = (127, 128) if d == 128 else (64, 72)
    edges = [0, 1, 7, 8, 16, 17, 63, 64] + ([65, 80, 100, 127] if d == 128 else [])
    lens = np.resize(np.array(edges, np.int32), B)
    e = _direct_case(B=B, Hk=Hk, Hv=Hv, d=d, Lmax=Lmax, cap=cap, in_dtype=in_dtype, seed=870 + B, lens=lens,
                     rec_dtype=rec_dtype, out_dtype=rec_dtype, block_size=block_size)
    say("buffer alone, B=%d heads %d/%d d=%d %s/%s: rel err out/u/decode/state %.2e %.2e %.2e %.2e" % ((B, Hk, Hv, d, in_dtype, rec_dtype) + e))
    # fp32: the state folded afterwards is a sum of up to 65 records, each off by 2^-24 of its size, and the error is
    # measured against an RMS that a quarter of the requests, with 0 or 1 record, pull down: the largest element is 13.5
    # times the RMS (d = 64) and 12.0 (d = 32) in the oracle's states
    H.check(e if in_dtype != "f32" else e[:3], in_dtype, rec_dtype, "buffer alone")
    assert in_dtype != "f32" or e[3] < 65 * 2.0 ** -24 * 13.6, e


@pytest.mark.parametrize("in_dtype, Lmax", [("bf16", 64), ("bf16", 128), ("f16", 128)])
def test_direct_products_of_full_fp32_factors(in_dtype, Lmax):
    """Outputs that are one product (q_i.k_0) u_0 of two factors with all 24 bits: three pieces to a factor, of whose nine
    products six are formed.  Rounded to nearest, the three that are left out are at most 5.4e-8 of the product (4 million
    pairs of normal values) and have no sign of their own; three sums in fp32 add 2^-24 each: 2.4e-7.  Cut off instead of
    rounded they are 4.3e-7, 4e-8 on the average."""
    rng = np.random.default_rng(880)
    Hk, Hv, d = 4, 8, 128
    tok = {x: np.zeros((1, Lmax, Hk if x in "qk" else Hv, d), np.float32) for x in "qkv"}
    tok["g"], tok["beta"] = np.zeros((1, Lmax, Hv), np.float32), np.zeros((1, Lmax, Hv), np.float32)

    def eight_bits(*size):   # 1 .. 2, exact in both types
        return (rng.integers(128, 256, size) / 128.0).astype(np.float32)
    # q.k = a c + b d: a c a multiple of 2^-14, b d one of 2^-22, their sum below 4
    tok["k"][0, 0, :, 0], tok["k"][0, 0, :, 1] = eight_bits(Hk), eight_bits(Hk) / 256
    tok["q"][0, :, :, 0], tok["q"][0, :, :, 1] = eight_bits(Lmax, Hk), eight_bits(Lmax, Hk)
    tok["v"][0, 0] = eight_bits(Hv, d) * rng.choice([-1, 1], (Hv, d))
    tok["beta"][0, 0] = rng.uniform(0.5, 1, Hv)
    lay = H.Layer(1, Hk, Hv, d, d, cap=Lmax, in_dtype=in_dtype, with_state=False)
    out = lay.new_out(1, Lmax, Hv, d, fill=float("nan"))
    lay.direct(H.dev(np.array([Lmax], np.int32)), Lmax, H.upload_tokens(tok, in_dtype), out)
    u0 = lay.u_records(0, 0, 1)[:, 0].astype(np.float64)                                          # [Hv, d]
    qk = (tok["q"][0].astype(np.float64) * tok["k"][0, 0].astype(np.float64)).sum(-1)             # [Lmax, Hk]
    want = np.repeat(qk, Hv // Hk, 1)[:, :, None] * u0
    e = (H.host(out)[0].astype(np.float64) - want) / want
    say("direct, full fp32 factors, %s Lmax=%d: error max %.2e mean %.2e" % (in_dtype, Lmax, np.abs(e).max(), e.mean()))
    assert np.abs(e).max() < 2.4e-7 and abs(e.mean()) < 1e-8, (np.abs(e).max(), e.mean())


@pytest.mark.parametrize("d, in_dtype, cap", [(128, "bf16", 16), (128, "f16", 64), (64, "bf16", 64), (128, "f32", 32)])
@pytest.mark.parametrize("Hk, Hv", [(1, 1), (2, 4)])
def test_fold_of_an_overdue_buffer(d, in_dtype, cap, Hk, Hv):
    """kvb_decode_flush whose threshold lies below, at and above the records that a request holds with its new token:
    every fill is a plain count again, and the state that a last kvb_flush completes is the recurrence's."""
    rng = np.random.default_rng(880 + cap + Hv)
    fills, C = np.array([0, 4, 5, 6, cap - 1, 3], np.int32), 6
    B, n = len(fills), int(fills.max()) + 1
    S0 = H.prefix_state(rng, B, Hk, Hv, d, d, in_dtype, 8)
    tok = synth.token_stream(rng, B, n, Hk, Hv, d, d, in_dtype)
    dtok = H.upload_tokens(tok, in_dtype)
    lay = H.Layer(B, Hk, Hv, d, d, cap, in_dtype)
    lay.set_state(S0)
    out = lay.new_out(B, Hv, d)
    for t in range(n - 1):   # request b joins so that all end at token n - 1
        who = np.flatnonzero(fills >= n - 1 - t)
        view = {x: y[torch.from_numpy(who).cuda(), t].contiguous() for x, y in dtok.items()}
        lay.decode(view, lay.new_out(len(who), Hv, d), slot=lay.slot[torch.from_numpy(who).cuda()].contiguous(), B=len(who))
    assert np.array_equal(lay.fill(), fills)
    lay.decode_flush(H.step_view(dtok, n - 1), out, C)
    assert np.array_equal(lay.fill(), np.where(fills + 1 >= C, 0, fills + 1))
    lay.flush(1)
    assert np.array_equal(lay.fill(), np.zeros(B, np.int32)) and not lay.status().any()
    errs = []
    for b in range(B):
        own = {x: y[b:b + 1, n - 1 - fills[b]:] for x, y in tok.items()}
        o, _, S, _ = oracle.gdn_sequence(S0[b:b + 1].astype(np.float64), own["q"], own["k"], own["v"], own["g"], own["beta"])
        errs += [H.rel_err(H.host(out[b]), o[0, -1]), H.rel_err(lay.get_state()[b], S[0])]
    say("overdue buffer, d=%d %s: rel err %.2e" % (d, in_dtype, max(errs)))
    H.check(errs, in_dtype, what="overdue buffer")


@pytest.mark.parametrize("d, Lmax, in_dtype", [(128, 128, "bf16"), (128, 64, "f16"), (64, 64, "bf16")])
@pytest.mark.parametrize("B, Hv", [(2, 256), (63, 9), (65, 8), (255, 3), (257, 2), (512, 1), (513, 1)])
def test_direct_longest_first(d, Lmax, in_dtype, B, Hv):
    """Batches around the wave, workgroup and table sizes of the sort by length, every class of lengths among them;
    an untaken unit leaves NaN in its outputs."""
    rng = np.random.default_rng(890 + B)
    lens = rng.integers(0, Lmax + 1, B).astype(np.int32)
    lens[:2] = [0, Lmax]
    e = _direct_case(B=B, Hk=1, Hv=Hv, d=d, Lmax=Lmax, cap=Lmax, in_dtype=in_dtype, seed=891 + B, lens=lens, then_decode=False)
    say("direct, longest first, d=%d B=%d: rel err out/u/decode/state %.2e %.2e %.2e %.2e" % ((d, B) + e))
    H.check(e, in_dtype, what="longest first")


SORTED_FORMS = [(128, 128, "f16", "f16", 16), (128, 128, "bf16", "f32", 8), (128, 64, "bf16", "bf16", 8), (128, 64, "f32", "f32", None),
                (128, 64, "f32", "f32", 16), (64, 64, "bf16", "f32", 8), (32, 64, "f16", "f16", None), (32, 64, "f32", "f32", 16)]


@pytest.mark.parametrize("d, Lmax, in_dtype, rec_dtype, block_size", SORTED_FORMS)
def test_direct_longest_first_forms(d, Lmax, in_dtype, rec_dtype, block_size):
    """The sorted launch with paged and 16-bit records, and in the block-row kernel, whose tables share its tiles."""
    B = 65
    lens = np.random.default_rng(895 + d).integers(0, Lmax + 1, B).astype(np.int32)
    e = _direct_case(B=B, Hk=4, Hv=8, d=d, Lmax=Lmax, cap=Lmax, in_dtype=in_dtype, seed=896 + d, lens=lens, then_decode=False,
                     rec_dtype=rec_dtype, out_dtype=rec_dtype, block_size=block_size, scatter=True)
    say("direct, longest first, d=%d %s/%s: rel err out/u/decode/state %.2e %.2e %.2e %.2e" % ((d, in_dtype, rec_dtype) + e))
    H.check(e, in_dtype, rec_dtype, "longest first")


@pytest.mark.parametrize("d, Lmax, in_dtype, rec_dtype, block_size", [SORTED_FORMS[i] for i in (1, 2, 3, 5, 6)])
def test_direct_longest_first_what_is_flagged(d, Lmax, in_dtype, rec_dtype, block_size):
    """Lengths outside 0..Lmax, sorted as the Lmax that they are clamped to and flagged, and slots outside the store, whose
    requests are skipped: each at its own place of the sorted order, with every other request as it should be."""
    B, Hk, Hv = 70, 4, 8
    rng = np.random.default_rng(897 + d + Lmax)
    lens = rng.integers(0, Lmax + 1, B).astype(np.int32)
    lens[[0, 17, 68]] = [-1, Lmax + 1, -2 ** 31]
    lens[[33, 64]] = [2 ** 31 - 1, 0]
    clamped = np.where((lens < 0) | (lens > Lmax), Lmax, lens).astype(np.int32)
    slots = rng.permutation(B).astype(np.int32)
    skipped = [5, 17, 69]
    slots[skipped] = [B, -1, 2 ** 31 - 1]
    tok = synth.token_stream(rng, B, Lmax, Hk, Hv, d, d, in_dtype)
    lay = H.Layer(B, Hk, Hv, d, d, Lmax, in_dtype, n_slots=B, slots=slots, with_state=False, rec_dtype=rec_dtype, out_dtype=rec_dtype,
                  block_size=block_size)
    lay.ds.fill.fill_(3)
    out = lay.new_out(B, Lmax, Hv, d, fill=float("nan"))
    lay.direct(H.dev(lens), Lmax, H.upload_tokens(tok, in_dtype), out)
    torch.cuda.synchronize()
    done = np.setdiff1d(np.arange(B), skipped)
    fill, status = np.full(B, 3, np.int32), np.zeros(B, np.int32)
    fill[slots[done]] = clamped[done]
    status[slots[done]] = np.where(lens[done] != clamped[done], 1, 0)   # KVB_STATUS_OVERFLOW
    assert np.array_equal(lay.ds.fill.cpu().numpy(), fill) and np.array_equal(lay.ds.status.cpu().numpy(), status)
    assert lay.spare_clean()
    ref, u_ref, _ = oracle.kvb_direct_expected(tok["q"], tok["k"], tok["v"], tok["g"], tok["beta"], clamped)
    ref[skipped] = np.nan
    got = H.host(out)
    valid = ~np.isnan(ref)
    assert np.array_equal(valid, ~np.isnan(got)), "what a request does not have was written, or what it has was not"
    errs = [H.rel_err(got[valid], ref[valid], lay.out_unit)]
    errs += [H.rel_err(lay.u_records(b, 0, clamped[b]).transpose(1, 0, 2), u_ref[b, :clamped[b]]) for b in done if clamped[b] > 0]
    say("direct, longest first, flagged, d=%d %s/%s: rel err %.2e" % (d, in_dtype, rec_dtype, max(errs)))
    H.check(errs, in_dtype, rec_dtype, "longest first, flagged")


@pytest.mark.parametrize("d, in_dtype, rec_dtype", [(128, i, r) for i, r in TYPES + [("f32", "f32")]]
                         + [(64, "bf16", "f32"), (64, "f32", "f32"), (32, "f16", "f16")])
@pytest.mark.parametrize("Hk, Hv, block_size", [(1, 2, None), (16, 48, None), (16, 32, 16)])
def test_buffer_step_blocks(d, in_dtype, rec_dtype, Hk, Hv, block_size):
    """kvb_decode without a state around every 16-record tile and 64-record block, with one and two v-heads a workgroup
    (and an odd head left over), contiguous and paged: the token that joins fills[b] records, and the record it leaves."""
    rng = np.random.default_rng(900 + d + Hv)
    fills = np.array([0, 1, 15, 16, 17, 63, 64, 65, 127], np.int32)
    B, n, cap = len(fills), 128, 128
    tok = synth.token_stream(rng, B, n, Hk, Hv, d, d, in_dtype)
    dtok = H.upload_tokens(tok, in_dtype)
    lay = H.Layer(B, Hk, Hv, d, d, cap, in_dtype, with_state=False, rec_dtype=rec_dtype, out_dtype=rec_dtype, block_size=block_size)
    for t in range(n - 1):   # request b joins so that all end at token n - 1
        who = torch.from_numpy(np.flatnonzero(fills >= n - 1 - t)).cuda()
        view = {x: y[who, t].contiguous() for x, y in dtok.items()}
        lay.decode(view, lay.new_out(len(who), Hv, d), slot=lay.slot[who].contiguous(), B=len(who))
    out = lay.new_out(B, Hv, d, fill=float("nan"))
    lay.decode(H.step_view(dtok, n - 1), out)
    torch.cuda.synchronize()
    assert np.array_equal(lay.fill(), fills + 1) and lay.spare_clean()
    errs = []
    for b in range(B):
        own = {x: y[b:b + 1, n - 1 - fills[b]:] for x, y in tok.items()}
        o, u, _, _ = oracle.gdn_sequence(np.zeros((1, Hv, d, d)), own["q"], own["k"], own["v"], own["g"], own["beta"])
        errs += [H.rel_err(H.host(out[b]), o[0, -1], lay.out_unit), H.rel_err(lay.u_records(b, 0, fills[b] + 1).transpose(1, 0, 2), u[0])]
    say("buffer step, d=%d %s/%s %d/%d heads: rel err %.2e" % (d, in_dtype, rec_dtype, Hk, Hv, max(errs)))
    H.check(errs, in_dtype, rec_dtype, "buffer step")


@pytest.mark.parametrize("d, in_dtype, rec_dtype, cap", [(128, i, r, 128) for i, r in TYPES] + [(128, "f32", "f32", 32), (64, "bf16", "f32", 128), (64, "f32", "f32", 48),
                                                         (32, "f16", "f16", 128)])
@pytest.mark.parametrize("block_size", [None, 16])
def test_buffer_step_two_heads(d, in_dtype, rec_dtype, cap, block_size):
    """kvb_decode without a state in launches that take two v-heads a workgroup (540 units, five v-heads to a key head, so that one
    is left over): around the tiles and blocks that cap holds, the token that joins fills[b] records, and the record it leaves."""
    rng = np.random.default_rng(950 + d)
    Hk, Hv, B = 2, 10, 54
    edges = [f for f in (0, 1, 15, 16, 17, 31, 47, 63, 64, 65, 127) if f < cap]
    fills = np.array([edges[b % len(edges)] for b in range(B)], np.int32)
    n = cap
    tok = synth.token_stream(rng, B, n, Hk, Hv, d, d, in_dtype)
    dtok = H.upload_tokens(tok, in_dtype)
    lay = H.Layer(B, Hk, Hv, d, d, cap, in_dtype, with_state=False, rec_dtype=rec_dtype, out_dtype=rec_dtype, block_size=block_size)
    for t in range(n - 1):   # request b joins so that all end at token n - 1
        who = torch.from_numpy(np.flatnonzero(fills >= n - 1 - t)).cuda()
        if len(who):
            view = {x: y[who, t].contiguous() for x, y in dtok.items()}
            lay.decode(view, lay.new_out(len(who), Hv, d), slot=lay.slot[who].contiguous(), B=len(who))
    out = lay.new_out(B, Hv, d, fill=float("nan"))
    lay.decode(H.step_view(dtok, n - 1), out)
    torch.cuda.synchronize()
    assert np.array_equal(lay.fill(), fills + 1) and lay.spare_clean()
    errs = []
    for b in range(len(edges)):
        own = {x: y[b:b + 1, n - 1 - fills[b]:] for x, y in tok.items()}
        o, u, _, _ = oracle.gdn_sequence(np.zeros((1, Hv, d, d)), own["q"], own["k"], own["v"], own["g"], own["beta"])
        errs += [H.rel_err(H.host(out[b]), o[0, -1], lay.out_unit), H.rel_err(lay.u_records(b, 0, fills[b] + 1).transpose(1, 0, 2), u[0])]
    say("buffer step, two heads, d=%d %s/%s: rel err %.2e" % (d, in_dtype, rec_dtype, max(errs)))
    H.check(errs, in_dtype, rec_dtype, "buffer step, two heads")


@pytest.mark.parametrize("in_dtype", ["bf16", "f16"])
def test_buffer_step_dots_add_pairwise(in_dtype):
    """kvb_decode without a state, delta values that pick one record each: its outputs are the dot products of the new query
    with the buffered keys.  128 positive terms, summed as 32, 64 and 128 of them: each level rounds by 0.289 units of at most
    2^-23 of its sums in the root mean square, and the sums of a level below count half as much and are twice as many."""
    d, Hk, Hv, B = 128, 2, 4, 48
    rng = np.random.default_rng(930)
    lay = H.Layer(B, Hk, Hv, d, d, 128, in_dtype, with_state=False)
    keys = np.abs(rng.standard_normal((B, Hk, 128, d)))
    lay.ds.buf_k.copy_(H.dev(keys.astype(np.float32), in_dtype))
    lay.ds.buf_u.copy_(torch.eye(128, device="cuda").expand(B, Hv, 128, d))
    lay.ds.fill.fill_(127)
    zeros = np.zeros((B, Hv), np.float32)
    tok = H.upload_tokens({"q": np.abs(rng.standard_normal((B, Hk, d))).astype(np.float32), "k": np.zeros((B, Hk, d), np.float32),
                           "v": np.zeros((B, Hv, d), np.float32), "g": zeros, "beta": zeros}, in_dtype)
    out = lay.new_out(B, Hv, d)
    lay.decode(tok, out)
    q, k = H.host(tok["q"]).astype(np.float64), H.host(lay.ds.buf_k).astype(np.float64)
    want = np.repeat(np.einsum("bhd,bhld->bhl", q, k), Hv // Hk, axis=1)[..., :127]
    err = np.linalg.norm(H.host(out)[..., :127] - want) / np.linalg.norm(want)
    say("dots of the buffer step, %s: rms error %.2e" % (in_dtype, err))
    assert err < 0.289 * 2.0 ** -23 * (1 + 1 / 2 + 1 / 4) ** 0.5, err
