"""Fill words in one array and with a 128-byte line to each slot (KVB_STORE_FILL_APART): every call that reads or changes
them leaves the same bits in both, whatever lies between the lines' first words, and finds slots by the stride it was told."""
import numpy as np
import pytest
import torch

import harness as H
from harness import oracle
from paper_2605_19049_amd import kvb, synth
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


def run(apart, in_dtype, rec_dtype, d, block_size, by_address):
    rng = np.random.default_rng(31 + d)
    B, Hk, Hv, C, T, n_slots = 7, 2, 6, 5, 3, 41
    lay = H.Layer(B, Hk, Hv, d, d, 16, in_dtype, n_slots=n_slots, slots=[40, 0, 33, 7, 32, 31, 1], rec_dtype=rec_dtype, out_dtype=rec_dtype,
                  block_size=block_size)
    ds = lay.ds
    rows = torch.full((n_slots, kvb.FILL_APART), -7, dtype=torch.int32, device="cuda")
    ds.fill = rows[:, 0] if apart else torch.empty(n_slots, dtype=torch.int32, device="cuda")
    ds.fill.fill_(2)   # (slots of no request keep it)
    ds.fill[lay.slot.long()] = 0
    flags = kvb.STORE_FILL_APART if apart else 0

    def st(state=True):   # the store by the fill tensor, or by its address and the flag
        return kvb.store(ds.state if state else None, ds.buf_k, ds.buf_u, ds.buf_G, ds.fill.data_ptr() if by_address else ds.fill, ds.status, n_slots,
                         flags if by_address else 0, ds.block_table, ds.block_size or 0, ds.max_blocks, ds.n_blocks)

    tok = H.upload_tokens(synth.token_stream(rng, B, 8, Hk, Hv, d, d, in_dtype), in_dtype)
    seen = []
    out = lay.new_out(B, 8, Hv, d, fill=0.0)
    lens = torch.tensor([8, 1, 0, 3, 7, 2, 5], dtype=torch.int32, device="cuda")
    acc = torch.tensor([0, 3, 1, 2, 3, 0, 1], dtype=torch.int32, device="cuda")
    sh = lay.shape()

    def after(name):
        torch.cuda.synchronize()
        seen.append((name, [x.clone() for x in (out, ds.state, ds.buf_k, ds.buf_u, ds.buf_G, ds.fill, ds.status)]))

    args = [tok[n] for n in ("q", "k", "v", "g", "beta")]
    kvb.kvb_direct(sh, st(False), lay.slot, lens, 8, *args, out)
    after("direct")
    step = [x[:, 0].contiguous() for x in args] + [lay.new_out(B, Hv, d, fill=0.0)]
    kvb.kvb_decode(sh, st(False), lay.slot, *step)
    after("decode without a state")
    kvb.kvb_flush(sh, st(), lay.slot, None, 1)
    after("fold")
    for i in range(6):
        kvb.kvb_decode_flush(sh, st(), lay.slot, *[x[:, i].contiguous() for x in args], step[-1], C)
    after("decode_flush")
    spec = [x[:, :T].contiguous() for x in args] + [lay.new_out(B, T, Hv, d, fill=0.0)]
    parent = torch.tensor([[-1, 0, 0]] * B, dtype=torch.int32, device="cuda")
    path = torch.tensor([[0, 2, 0]] * B, dtype=torch.int32, device="cuda")
    kvb.kvb_verify_tree(sh, st(), lay.slot, T, parent, *spec)
    kvb.kvb_compact(sh, st(), lay.slot, T, path, acc.clamp(max=2))
    kvb.kvb_flush(sh, st(), lay.slot, acc.clamp(max=2), C)
    after("tree")
    kvb.kvb_verify(sh, st(), lay.slot, T, *spec)
    kvb.kvb_flush(sh, st(), lay.slot, acc, C)
    kvb.kvb_decode(sh, st(), lay.slot, *step)
    after("verify, commit, decode")
    if apart:
        assert bool((rows[:, 1:] == -7).all())
    others = torch.ones(n_slots, dtype=torch.bool)
    others[lay.slots_np] = False
    assert bool((ds.fill.cpu()[others] == 2).all()) and not ds.status.any()
    return seen


@pytest.mark.parametrize("in_dtype, rec_dtype, d, block_size", [("bf16", "f32", 128, None), ("f16", "f16", 128, 8), ("f32", "f32", 64, None)])
def test_fill_words_apart(in_dtype, rec_dtype, d, block_size):
    packed = run(False, in_dtype, rec_dtype, d, block_size, False)
    for by_address in (False, True):
        apart = run(True, in_dtype, rec_dtype, d, block_size, by_address)
        for (name, a), (_, b) in zip(packed, apart):
            assert all(torch.equal(x, y) for x, y in zip(a, b)), name


@pytest.mark.parametrize("d, in_dtype, rec_dtype, B", [(64, "bf16", "f32", 18), (32, "f32", "f32", 17), (128, "f32", "f32", 44), (128, "bf16", "f32", 44), (128, "f16", "f16", 90),
                                                        (64, "bf16", "f32", 90), (64, "f32", "f32", 90)])
@pytest.mark.parametrize("apart", [False, True])
def test_launches_that_the_layout_decides(d, in_dtype, rec_dtype, B, apart):
    """Sizes at which the layouts differ in the v-heads a workgroup takes (kvb_decode without a state, 102 to 264 units) or in how
    units are dealt (540): a context decoded from the buffer alone, folded, and decoded on with folds, against the recurrence."""
    rng = np.random.default_rng(61 + B)
    Hk, Hv, n, C = 2, 6, 6, 4
    lay = H.Layer(B, Hk, Hv, d, d, 128, in_dtype, scale=d ** -0.5, n_slots=B + 9, slots=rng.permutation(B + 9)[:B], rec_dtype=rec_dtype, out_dtype=rec_dtype)
    if not apart:
        lay.ds.fill = torch.zeros(B + 9, dtype=torch.int32, device="cuda")
    tok = synth.token_stream(rng, B, 2 * n, Hk, Hv, d, d, in_dtype)
    dtok = H.upload_tokens(tok, in_dtype)
    out = lay.new_out(B, 2 * n, Hv, d, fill=float("nan"))
    for t in range(2 * n):
        o = lay.new_out(B, Hv, d, fill=float("nan"))
        if t < n:
            lay.decode(H.step_view(dtok, t), o, use_state=False)
        else:
            lay.decode_flush(H.step_view(dtok, t), o, C)
        if t == n - 1:
            lay.flush(1)
        out[:, t] = o
    torch.cuda.synchronize()
    assert bool((lay.fill() == n % C).all()) and not lay.status().any() and int(lay.ds.fill.sum()) == B * (n % C)
    ref, _, _ = oracle.kvb_decode_expected(np.zeros((B, Hv, d, d)), tok["q"], tok["k"], tok["v"], tok["g"], tok["beta"], scale=d ** -0.5)
    e = H.rel_err(H.host(out), ref, lay.out_unit)
    say("%s fill words, d=%d %s/%s B=%d: rel err %.2e" % ("apart" if apart else "packed", d, in_dtype, rec_dtype, B, e))
    H.check([e], in_dtype, rec_dtype, "fill layout")


@pytest.mark.parametrize("in_dtype, rec_dtype", [("bf16", "f32"), ("f16", "f16"), ("f32", "f32")])
@pytest.mark.parametrize("B, threshold, commit", [(33, 1, False), (64, 1, False), (96, 1, False), (96, 1, True), (192, 2, True), (480, 1, True)])
def test_folds_of_whole_batches(in_dtype, rec_dtype, B, threshold, commit):
    """kvb_flush where all requests fold, or nearly, at the sizes where states are stored plainly (264 to 512 units), where units are
    no longer dealt for it and where they are again: a request is folded to the same bits as in smaller launches."""
    rng = np.random.default_rng(B + threshold)
    Hk, Hv, d, cap = 4, 8, 128, 16
    lay = H.Layer(B, Hk, Hv, d, d, cap, in_dtype, n_slots=B + 5, slots=rng.permutation(B + 5)[:B], rec_dtype=rec_dtype)
    ds = lay.ds
    ds.state.normal_(0, 0.5)
    ds.buf_u.copy_(torch.randn(ds.buf_u.shape, device="cuda"))
    ds.buf_k.copy_(torch.nn.functional.normalize(torch.randn(ds.buf_k.shape, device="cuda"), dim=-1))
    ds.buf_G.copy_(-0.25 * torch.arange(1, cap + 1, device="cuda").float().expand_as(ds.buf_G))
    fills = torch.from_numpy(rng.integers(0, cap - 3, B).astype(np.int32)).cuda()
    acc = torch.from_numpy(rng.integers(0, 4, B).astype(np.int32)).cuda() if commit else None
    state = ds.state.clone()
    seen = []
    few = 32 if B <= 64 else 64
    for parts in ([(0, B)], [(b, min(b + few, B)) for b in range(0, B, few)]):
        ds.state.copy_(state)
        ds.fill.fill_(7)
        ds.fill[lay.slot.long()] = fills
        for lo, hi in parts:
            kvb.kvb_flush(lay.shape(hi - lo), ds.c(), lay.slot[lo:hi].contiguous(), None if acc is None else acc[lo:hi].contiguous(), threshold)
        torch.cuda.synchronize()
        seen.append((ds.state.clone(), ds.fill.clone()))
    due = (fills if acc is None else fills + acc) >= threshold
    assert bool((seen[0][1][lay.slot.long()] == torch.where(due, 0, fills if acc is None else fills + acc)).all()) and not ds.status.any()
    assert all(torch.equal(x, y) for x, y in zip(*seen)) and not torch.equal(seen[0][0], state)


def test_device_store_keeps_a_line_to_each_slot():
    ds = kvb.DeviceStore(3, 1, 2, 32, 32, 8, kvb.F32)
    assert ds.fill.shape == (3,) and ds.fill.stride() == (kvb.FILL_APART,) and ds.fill.data_ptr() % 128 == 0
    assert ds.c().flags == kvb.STORE_FILL_APART and ds.c(flags=kvb.STORE_STREAM).flags == kvb.STORE_FILL_APART | kvb.STORE_STREAM
