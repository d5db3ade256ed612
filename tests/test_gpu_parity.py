"""GPU parity: the HIP library, called through the C ABI, against the CPU oracle on the same
seeded inputs.  bf16 path: max abs error 2e-2 on the fp32-stored block outputs; fp32 path:
1e-3 relative; integer logic (sync counts, rank indexing) bit-exact."""
import dataclasses

import numpy as np
import pytest

from oracle import spd_oracle as O
from paper_2502_20727_amd import binding as B
from paper_2502_20727_amd import inputs, workloads
from paper_2502_20727_amd.workloads import BF16, F32, Workload

from helpers import Case, assert_close, cache_storage, oracle_shapes

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


# ------------------------------------------------------------------------------------------------
# rank-sum: the kept sync point
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("n_slots,n,with_base", [(0, 64, True), (1, 7, True), (2, 1024, False), (8, 4099, True),
                                                 (8, 16 * 8192, True), (3, 1, False)])
def test_rank_sum(gpu, n_slots, n, with_base):
    import torch
    ctx = B.spd_create(B.make_config(workloads.TOY, max_ctx=64))
    rng = np.random.default_rng(n_slots * 1000 + n)
    slots = rng.standard_normal((max(n_slots, 1), n)).astype(np.float32)
    base = rng.standard_normal(n).astype(np.float32) if with_base else None
    d_slots = torch.from_numpy(slots).to(gpu)
    d_base = torch.from_numpy(base).to(gpu) if with_base else None
    out = torch.full((n,), 7.0, dtype=torch.float32, device=gpu)
    B.spd_rank_sum(ctx, d_base, d_slots, n_slots, n, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    # contract: partials in ascending slot order, base last, all in fp32 -> bit-exact
    acc = np.zeros(n, np.float32)
    if n_slots:
        acc = slots[0].copy()
        for s in range(1, n_slots):
            acc = acc + slots[s]
    want32 = (base + acc) if with_base else acc
    assert np.array_equal(got, want32.astype(np.float32))
    want64 = O.rank_sum(base, slots[:n_slots]) if n_slots else (np.asarray(base, np.float64) if with_base else np.zeros(n))
    assert np.max(np.abs(got - want64)) <= 1e-5 * max(1.0, float(np.max(np.abs(want64))))
    B.spd_destroy(ctx)


# ------------------------------------------------------------------------------------------------
# configuration 0: the fp32 toy model, all ranks emulated, prefill 32 + 8 single-token steps
# ------------------------------------------------------------------------------------------------
def test_toy_fp32_prefill_then_decode(gpu):
    import torch
    w = workloads.TOY
    case = Case(w, gpu, ranks=range(w.tp), positions=[0], max_ctx=64, max_tokens=32)
    X = inputs.hidden_states(w, 40)
    slots = torch.zeros((w.tp, 32, w.hidden), dtype=torch.float32, device=gpu)
    out = torch.empty((32, w.hidden), dtype=torch.float32, device=gpu)
    syncs = B.spd_model_forward(case.dev.ctx, w.mask, B.SPD_ALL_RANKS, case.dev.weights, case.dev.kv, [0], 1, 32,
                                case.to_dev(X[:32]), slots, out, case.dev.workspace)
    torch.cuda.synchronize()
    want, osyncs = O.model_all_ranks(case.sh, X[:32], case.shards, case.caches, [0], 1, 32, w.mask)
    assert syncs == osyncs == 3                        # mask [1, 0]: 1 + 2 sync points
    err = assert_close(out.cpu().numpy(), want, w, "toy prefill")
    say(f"toy prefill: max err {err:.2e}, max |oracle| {np.max(np.abs(want)):.2f}")
    for t in range(32, 40):                            # teacher-forced single-token steps
        o1 = torch.empty((1, w.hidden), dtype=torch.float32, device=gpu)
        B.spd_model_forward(case.dev.ctx, w.mask, B.SPD_ALL_RANKS, case.dev.weights, case.dev.kv, [t], 1, 1,
                            case.to_dev(X[t:t + 1]), slots, o1, case.dev.workspace)
        torch.cuda.synchronize()
        want, _ = O.model_all_ranks(case.sh, X[t:t + 1], case.shards, case.caches, [t], 1, 1, w.mask)
        assert_close(o1.cpu().numpy(), want, w, f"toy decode step {t}")
    case.close()


def _block_with_taps(case, li, flag, rank_arg, x_dev, slots, batch, q_len, positions):
    import torch
    w = case.w
    M = batch * q_len
    qd = w.q_per_rank * w.head_dim
    taps = dict(q=torch.zeros((M, qd), dtype=torch.float32, device=x_dev.device),
                attn=torch.zeros((M, qd), dtype=torch.float32, device=x_dev.device),
                y=torch.zeros((M, w.hidden), dtype=torch.float32, device=x_dev.device),
                u=torch.zeros((M, w.ffn_per_rank), dtype=torch.float32, device=x_dev.device))
    out = torch.empty((M, w.hidden), dtype=torch.float32, device=x_dev.device)
    B.spd_block_forward(case.dev.ctx, li, flag, rank_arg, case.dev.weights[li], case.dev.kv[li], positions, batch,
                        q_len, x_dev, slots, out, case.dev.workspace, taps=taps)
    torch.cuda.synchronize()
    return out, {k: v.cpu().numpy() for k, v in taps.items()}


def _check_taps(taps, det, w, what):
    # bf16-stored intermediates carry one rounding of their own: half an ulp (2^-9 relative) on top
    for name, key in (("q", "Q"), ("attn", "A"), ("y", "Y"), ("u", "U")):
        want = det[key]
        scale = 1.0 + float(np.max(np.abs(want))) * (2.0 ** -8) / 2e-2 if w.dtype == BF16 else 1.0
        assert_close(taps[name], want, w, f"{what} tap {name}", scale=scale)


def test_toy_fp32_block_intermediates(gpu):
    import torch
    w = workloads.TOY
    for flag in (1, 0):
        case = Case(w, gpu, ranks=range(w.tp), positions=[0], max_ctx=64, max_tokens=32)
        X = inputs.hidden_states(w, 32)
        slots = torch.zeros((w.tp, 32, w.hidden), dtype=torch.float32, device=gpu)
        out, taps = _block_with_taps(case, 0, flag, B.SPD_ALL_RANKS, case.to_dev(X), slots, 1, 32, [0])
        det = {}
        want, _ = O.block_all_ranks(case.sh, X, case.shards[0], case.caches[0], [0], 1, 32, flag, det)
        assert_close(out.cpu().numpy(), want, w, f"toy block flag={flag}")
        # the taps belong to the last rank run
        d2 = {}
        c2 = O.KVCache(1, w.kv_per_rank, 64, w.head_dim)
        r = w.tp - 1
        Y = O.attention_partial(case.sh, X, case.shards[0][r], c2, [0], 1, 32, detail=d2)
        R = X + (Y if flag else sum(det["Y"]))
        O.mlp_partial(case.sh, R, case.shards[0][r], d2)
        d2["Y"] = Y
        _check_taps(taps, d2, w, f"toy flag={flag}")
        # slots hold what meets at the final sync point
        got_slots = slots.cpu().numpy()
        for i in range(w.tp):
            assert_close(got_slots[i], det["P"][i], w, f"toy slot {i} flag={flag}")
        case.close()


# ------------------------------------------------------------------------------------------------
# bf16 path, small shapes, all ranks: several tiles, ragged tails, ragged positions
# ------------------------------------------------------------------------------------------------
SMALL = Workload(name="small-bf16", hidden=256, n_q_heads=8, n_kv_heads=4, head_dim=64, ffn=832, n_layers=2,
                 tp=4, dtype=BF16, seed=11, batch=3, q_len=1, ctx=64, mask=(1, 0))
SMALL_MHA = Workload(name="small-bf16-mha", hidden=128, n_q_heads=4, n_kv_heads=4, head_dim=128, ffn=256,
                     n_layers=1, tp=2, dtype=BF16, seed=12, batch=2, q_len=1, ctx=64, mask=(1,))


# 3200 FFN columns per rank: 200 tiles of 16 do not fill the chip evenly, so decode-sized calls read the
# copy of the gate/up weights with 13-column groups (247 groups, the last one with 2 real columns)
NARROW_GU = Workload(name="narrow-gate-up", hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=6400, n_layers=1,
                     tp=2, dtype=BF16, seed=14, batch=3, q_len=1, ctx=64, mask=(1,))


# 2080 FFN columns per rank (130 pairs of gate/up tiles, no whole number of GEMM tiles) and 37 k-tiles (the last step
# of two holds one): gate/up takes K slices of the LDS-tiled GEMM at 65 .. 128 tokens, the skinny kernel at 17 .. 64 and beyond
WIDE_MID = Workload(name="wide-ffn-mid", hidden=1184, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=4160, n_layers=1,
                    tp=2, dtype=BF16, seed=17, batch=2, q_len=1, ctx=64, mask=(1,))


# head sizes other than LLaMA2's 128 and the small shapes' 64: 96 (six 16-wide slices per head, three rotary tile
# pairs) and 32 (two slices), with grouped KV heads
SMALL_D96 = Workload(name="small-bf16-d96", hidden=256, n_q_heads=8, n_kv_heads=4, head_dim=96, ffn=512, n_layers=1,
                     tp=2, dtype=BF16, seed=21, batch=3, q_len=1, ctx=64, mask=(1,))
SMALL_D32 = Workload(name="small-bf16-d32", hidden=128, n_q_heads=8, n_kv_heads=2, head_dim=32, ffn=256, n_layers=1,
                     tp=2, dtype=BF16, seed=22, batch=3, q_len=1, ctx=64, mask=(1,))


@pytest.mark.parametrize("w", [SMALL, SMALL_MHA, NARROW_GU, WIDE_MID, SMALL_D96, SMALL_D32], ids=lambda w: w.name)
@pytest.mark.parametrize("batch,q_len,positions", [
    (3, 1, [0, 17, 40]),          # decode, ragged contexts, one sequence with a single key
    (2, 7, [0, 5]),               # 14 tokens: a partial m-tile
    (2, 10, [0, 4]),              # 20 tokens: two m-tiles
    (3, 11, [3, 0, 20]),          # 33 tokens: three m-tiles with a ragged tail
    (1, 40, [8]),                 # one long chunk crossing several key blocks
    (2, 50, [0, 5]),              # 100 tokens: seven m-tiles, the last one ragged
    (3, 50, [0, 5, 14]),          # 150 tokens: two groups of 8 m-tiles per projection, the second one partly empty
], ids=["decode", "chunk14", "chunk20", "chunk33", "chunk40", "chunk100", "chunk150"])
@pytest.mark.parametrize("flag", [1, 0], ids=["spd", "tp"])
def test_bf16_small_all_ranks(gpu, w, batch, q_len, positions, flag):
    import torch
    M = batch * q_len
    case = Case(w, gpu, ranks=range(w.tp), positions=positions, max_ctx=64, max_tokens=max(48, M))
    X = inputs.hidden_states(w, M)
    slots = torch.zeros((w.tp, M, w.hidden), dtype=torch.float32, device=gpu)
    say(f"case {w.name} batch={batch} q_len={q_len} pos={positions} flag={flag}")
    out, taps = _block_with_taps(case, 0, flag, B.SPD_ALL_RANKS, case.to_dev(X), slots, batch, q_len, positions)
    det = {}
    want, _ = O.block_all_ranks(case.sh, X, case.shards[0], case.caches[0], positions, batch, q_len, flag, det)
    r = w.tp - 1
    d2 = {}
    c2 = O.KVCache(batch, w.kv_per_rank, 64, w.head_dim, storage=cache_storage(w))
    c2.k[...] = 0
    # the last rank's intermediates: recompute them with a cache holding the same prefill
    if max(positions) > 0:
        k, v = inputs.kv_prefill(w, 0, r, batch, max(positions))
        for b, p in enumerate(positions):
            k[b, :, p:, :] = 0.0
            v[b, :, p:, :] = 0.0
        c2.fill(k, v)
    Y = O.attention_partial(case.sh, X, case.shards[0][r], c2, positions, batch, q_len, detail=d2)
    O.mlp_partial(case.sh, X + (Y if flag else sum(det["Y"])), case.shards[0][r], d2)
    d2["Y"] = Y
    _check_taps(taps, d2, w, "small")
    err = assert_close(out.cpu().numpy(), want, w, "small block output")
    say(f"  block output max err {err:.2e} (max |oracle| {np.max(np.abs(want)):.2f})")
    # the appended keys / values: bf16 copies of the oracle's
    for i, rr in enumerate(case.ranks):
        n_pos = max(positions) + q_len
        k, v = case.dev.read_kv(0, i, batch, n_pos)
        for b, p in enumerate(positions):
            ko, vo = case.caches[0][i].k[b, :, p:p + q_len], case.caches[0][i].v[b, :, p:p + q_len]
            # both sides hold bf16 values; a last-bit disagreement is one ulp (2^-7 relative at most)
            assert np.max(np.abs(k[b, :, p:p + q_len] - ko)) <= 2.0 ** -7 * np.max(np.abs(ko)) + 1e-3
            assert np.max(np.abs(v[b, :, p:p + q_len] - vo)) <= 2.0 ** -7 * np.max(np.abs(vo)) + 1e-3
    case.close()


SMALL_H512 = Workload(name="small-bf16-h512", hidden=512, n_q_heads=8, n_kv_heads=4, head_dim=64, ffn=832, n_layers=1,
                      tp=4, dtype=BF16, seed=18, batch=3, q_len=1, ctx=64, mask=(1,))


@pytest.mark.parametrize("w", [SMALL, SMALL_H512, SMALL_MHA, SMALL_D96, SMALL_D32], ids=lambda w: w.name)
@pytest.mark.parametrize("flag", [1, 0], ids=["spd", "tp"])
@pytest.mark.parametrize("split", [B.SPD_SPLIT_AUTO, B.SPD_SPLIT_ALWAYS, B.SPD_SPLIT_NEVER], ids=["default", "all-split", "no-split"])
def test_bf16_long_call_small_shape(gpu, w, flag, split):
    """More than 512 tokens in one call on a small shape, all ranks: the launch shapes of the long
    prefill (LDS-tiled GEMM, key-split attention, row-wise norm preparation) with a ragged last
    m-tile, every output element checked (hidden size 256 and 512: one and two pieces of 256 features per
    workgroup of the row-wise preparation; the 128-wide shape takes the 256 x 256 tiles with their block-wise
    numbering, most of whose blocks stick out of so small a matrix)."""
    import torch
    batch, q_len, positions = 3, 181, [0, 0, 0]          # 543 tokens = 33 m-tiles + 15 rows
    M = batch * q_len
    case = Case(w, gpu, ranks=range(w.tp), positions=positions, max_ctx=192, max_tokens=M, act_split=split)
    X = inputs.hidden_states(w, M)
    slots = torch.zeros((w.tp, M, w.hidden), dtype=torch.float32, device=gpu)
    say(f"long call on the small shape: {M} tokens flag={flag} split={split}")
    out = torch.empty((M, w.hidden), dtype=torch.float32, device=gpu)
    B.spd_block_forward(case.dev.ctx, 0, flag, B.SPD_ALL_RANKS, case.dev.weights[0], case.dev.kv[0], positions, batch,
                        q_len, case.to_dev(X), slots, out, case.dev.workspace)
    torch.cuda.synchronize()
    want, _ = O.block_all_ranks(case.sh, X, case.shards[0], case.caches[0], positions, batch, q_len, flag, {})
    err = assert_close(out.cpu().numpy(), want, w, "long call block output")
    say(f"  block output max err {err:.2e} (max |oracle| {np.max(np.abs(want)):.2f})")
    case.close()


# contraction lengths at which the LDS-tiled GEMM can go wrong: fewer k-tiles than it has stages (one k-tile in the O
# projection, three in QKV and gate/up), odd numbers of them (down: 23), K slices of uneven lengths (66 k-tiles in 8
# slices), and 66 partial sums of squares per token, which a kernel of its own
# adds up before the gate/up projection of an SPD block of more than 512 tokens
KT_FEW = Workload(name="few-k-tiles", hidden=96, n_q_heads=2, n_kv_heads=2, head_dim=32, ffn=96, n_layers=1, tp=2, dtype=BF16,
                  seed=31, batch=1, q_len=1, ctx=64, mask=(1,))
KT_ODD = Workload(name="odd-k-tiles", hidden=2112, n_q_heads=4, n_kv_heads=2, head_dim=32, ffn=1440, n_layers=1, tp=2,
                  dtype=BF16, seed=32, batch=1, q_len=1, ctx=64, mask=(1,))


@pytest.mark.parametrize("w", [KT_FEW, KT_ODD], ids=lambda w: w.name)
@pytest.mark.parametrize("flag", [1, 0], ids=["spd", "tp"])
@pytest.mark.parametrize("split", [B.SPD_SPLIT_AUTO, B.SPD_SPLIT_ALWAYS, B.SPD_SPLIT_NEVER], ids=["default", "all-split", "no-split"])
@pytest.mark.parametrize("q_len", [17, 64, 100, 145, 384, 513, 530])
def test_bf16_gemm_contraction_lengths(gpu, w, flag, split, q_len):
    import torch
    case = Case(w, gpu, ranks=range(w.tp), positions=[0], max_ctx=544, max_tokens=q_len, act_split=split)
    X = inputs.hidden_states(w, q_len)
    slots = torch.zeros((w.tp, q_len, w.hidden), dtype=torch.float32, device=gpu)
    say(f"contraction lengths: {w.name} {q_len} tokens flag={flag} split={split}")
    out = torch.empty((q_len, w.hidden), dtype=torch.float32, device=gpu)
    B.spd_block_forward(case.dev.ctx, 0, flag, B.SPD_ALL_RANKS, case.dev.weights[0], case.dev.kv[0], [0], 1, q_len,
                        case.to_dev(X), slots, out, case.dev.workspace)
    torch.cuda.synchronize()
    want, _ = O.block_all_ranks(case.sh, X, case.shards[0], case.caches[0], [0], 1, q_len, flag, {})
    err = assert_close(out.cpu().numpy(), want, w, "block output")
    say(f"  block output max err {err:.2e} (max |oracle| {np.max(np.abs(want)):.2f})")
    case.close()


# 128 x 192 tiles begin in the middle of a group of eight m-tiles: last tiles of 1, 2, 5 and 12 m-tiles in the O projection, which is never
# sliced beyond 512 tokens (66 pairs of n-tiles), with fewer k-tiles than stages (2) and several turns of them, odd and even (15, 16)
def _long_o(heads):
    return Workload(name=f"o-{heads}-k-tiles", hidden=2112, n_q_heads=2 * heads, n_kv_heads=2, head_dim=32, ffn=128, n_layers=1, tp=2, dtype=BF16,
                    seed=56, batch=1, q_len=1, ctx=64, mask=(1,))


@pytest.mark.parametrize("w", [KT_ODD, _long_o(15), _long_o(16)], ids=lambda w: w.name)
@pytest.mark.parametrize("split", [B.SPD_SPLIT_AUTO, B.SPD_SPLIT_ALWAYS], ids=["default", "all-split"])
@pytest.mark.parametrize("q_len", [577, 608, 656, 768])
def test_bf16_gemm_tiles_across_groups(gpu, w, split, q_len):
    _one_rank_block(gpu, w, 1, q_len, [0], q_len % 2, split)


# 65 partial sums of squares per token after a kept attention sync point of more than 512 tokens (hidden sizes that the row-wise
# and the tile-wise preparation kernel serve): one preparation for all emulated ranks, whose partial sums every rank's
# gate/up projection needs whole
ROWS_65 = Workload(name="65-partials-rows", hidden=16640, n_q_heads=2, n_kv_heads=2, head_dim=32, ffn=2048, n_layers=1, tp=2, dtype=BF16,
                   seed=33, batch=1, q_len=1, ctx=64, mask=(0,))
TILES_65 = Workload(name="65-partials-tiles", hidden=16416, n_q_heads=2, n_kv_heads=2, head_dim=32, ffn=2048, n_layers=1, tp=2, dtype=BF16,
                    seed=34, batch=1, q_len=1, ctx=64, mask=(0,))


@pytest.mark.parametrize("w", [ROWS_65, TILES_65], ids=lambda w: w.name)
@pytest.mark.parametrize("flag", [1, 0], ids=["spd", "tp"])
def test_bf16_norm_partials_serve_every_rank(gpu, w, flag):
    import torch
    q_len = 513
    case = Case(w, gpu, ranks=range(w.tp), positions=[0], max_ctx=544, max_tokens=q_len)
    X = inputs.hidden_states(w, q_len)
    slots = torch.zeros((w.tp, q_len, w.hidden), dtype=torch.float32, device=gpu)
    say(f"norm partials: {w.name} flag={flag}")
    out = torch.empty((q_len, w.hidden), dtype=torch.float32, device=gpu)
    B.spd_block_forward(case.dev.ctx, 0, flag, B.SPD_ALL_RANKS, case.dev.weights[0], case.dev.kv[0], [0], 1, q_len,
                        case.to_dev(X), slots, out, case.dev.workspace)
    torch.cuda.synchronize()
    det = {}
    want, _ = O.block_all_ranks(case.sh, X, case.shards[0], case.caches[0], [0], 1, q_len, flag, det)
    got = slots.cpu().numpy().astype(np.float64)
    # a partial lost moves the factor by 1/130 and Z by twice that; fp16 operands leave 2^-11 each: 4 operands, 4 x 2^-11 at most
    for r in range(w.tp):
        err = float(np.linalg.norm(got[r] - det["P"][r]) / np.linalg.norm(det["P"][r]))
        say(f"  slot {r}: relative error {err:.2e}")
        assert err <= 4 * 2.0 ** -11, (r, err)
    case.close()


def _one_rank_block(gpu, w, batch, q_len, positions, flag, split=B.SPD_SPLIT_AUTO, max_ctx=None, bias_std=0.0, bound_scale=1.0, rank=1):
    """One rank's block call with peer slots as inputs against the oracle: the output, the slot the rank wrote, and the
    peers' slots unchanged."""
    import torch
    M = batch * q_len
    case = Case(w, gpu, ranks=[rank], positions=positions, max_ctx=max_ctx or (max(positions) + q_len + 31) // 32 * 32, max_tokens=M,
                act_split=split, bias_std=bias_std)
    X = inputs.hidden_states(w, M)
    peers = inputs.peer_slots(w, M)
    slots = case.to_dev(peers).reshape(w.tp, M, w.hidden)
    say(f"one rank: {w.name} {batch} x {q_len} tokens flag={flag} split={split}")
    out = torch.empty((M, w.hidden), dtype=torch.float32, device=gpu)
    B.spd_block_forward(case.dev.ctx, 0, flag, rank, case.dev.weights[0], case.dev.kv[0], positions, batch, q_len, case.to_dev(X),
                        slots, out, case.dev.workspace)
    torch.cuda.synchronize()
    o_slots = peers.astype(np.float64).reshape(w.tp, M, w.hidden)
    want = O.block_single_rank(case.sh, X, case.shards[0][0], case.caches[0][0], positions, batch, q_len, flag, rank, o_slots)
    err = assert_close(out.cpu().numpy(), want, w, "block output", scale=bound_scale)
    got = slots.cpu().numpy()
    assert_close(got[rank], o_slots[rank], w, "own slot", scale=bound_scale)
    for r in range(w.tp):
        if r != rank:
            assert np.array_equal(got[r], peers.reshape(w.tp, M, w.hidden)[r])
    say(f"  block output max err {err:.2e} (max |oracle| {np.max(np.abs(want)):.2f})")
    case.close()


# the kernel that streams a large gate/up matrix for up to 128 tokens, at its edges: 194 pairs of n-tiles (24 groups of
# eight and one with six spare waves) x 255 k-tiles (the last stage of two holds one)
MID_EDGE = Workload(name="mid-edges", hidden=8160, n_q_heads=2, n_kv_heads=2, head_dim=32, ffn=6208, n_layers=1, tp=2, dtype=BF16,
                    seed=35, batch=1, q_len=1, ctx=64, mask=(1,))


# ... and the medium one that it serves beyond 64 tokens: 130 pairs x 159 k-tiles
MID_LONG_EDGE = Workload(name="mid-long-edges", hidden=5088, n_q_heads=2, n_kv_heads=2, head_dim=32, ffn=4160, n_layers=1, tp=2, dtype=BF16,
                         seed=42, batch=1, q_len=1, ctx=64, mask=(1,))


@pytest.mark.parametrize("w", [MID_EDGE, MID_LONG_EDGE], ids=lambda w: w.name)
@pytest.mark.parametrize("q_len,flag", [(17, 1), (64, 0), (65, 0), (100, 1), (128, 0)])
def test_bf16_large_gate_up_short_call(gpu, w, q_len, flag):
    _one_rank_block(gpu, w, 1, q_len, [0], flag)


# decode QKV projections that K slices or one whole contraction could serve: 96 pairs of n-tiles (from which a
# contraction of 32 .. 64 k-tiles is done whole in the other projections), 64 and 32 k-tiles, up to four m-tiles
QKV_96 = Workload(name="qkv-96-pairs", hidden=2048, n_q_heads=16, n_kv_heads=16, head_dim=128, ffn=256, n_layers=1, tp=2, dtype=BF16,
                  seed=36, batch=1, q_len=1, ctx=64, mask=(1,))
QKV_96_SHORT = Workload(name="qkv-96-pairs-short", hidden=1024, n_q_heads=32, n_kv_heads=32, head_dim=64, ffn=256, n_layers=1, tp=2,
                        dtype=BF16, seed=37, batch=1, q_len=1, ctx=64, mask=(1,))


@pytest.mark.parametrize("w", [QKV_96, QKV_96_SHORT], ids=lambda w: w.name)
@pytest.mark.parametrize("split", [B.SPD_SPLIT_AUTO, B.SPD_SPLIT_ALWAYS], ids=["default", "all-split"])
@pytest.mark.parametrize("batch", [1, 3, 16, 17, 40, 64])
def test_bf16_decode_qkv_of_medium_width(gpu, w, split, batch):
    positions = [(7 * i) % 61 for i in range(batch)]
    _one_rank_block(gpu, w, batch, 1, positions, batch % 2, split, max_ctx=64)


# projections on either side of the lines between the skinny kernel and K slices: 101 k-tiles (slices of all tile shapes in
# QKV and gate/up; odd), 65 in down (skinny beyond 128 tokens, slices beyond 256), and 63 .. 65 of them at 33 .. 128 tokens
KT_101 = Workload(name="101-k-tiles", hidden=3232, n_q_heads=8, n_kv_heads=4, head_dim=32, ffn=4160, n_layers=1, tp=2, dtype=BF16,
                  seed=38, batch=1, q_len=1, ctx=64, mask=(1,))
KT_64 = Workload(name="64-k-tiles", hidden=2048, n_q_heads=20, n_kv_heads=4, head_dim=64, ffn=1600, n_layers=1, tp=2, dtype=BF16,
                 seed=39, batch=1, q_len=1, ctx=64, mask=(1,))


@pytest.mark.parametrize("w", [KT_101, KT_64], ids=lambda w: w.name)
@pytest.mark.parametrize("split", [B.SPD_SPLIT_AUTO, B.SPD_SPLIT_ALWAYS, B.SPD_SPLIT_NEVER], ids=["default", "all-split", "no-split"])
@pytest.mark.parametrize("q_len", [17, 32, 33, 64, 65, 128, 129, 256, 257, 512])
def test_bf16_short_and_sliced_contractions(gpu, w, split, q_len):
    _one_rank_block(gpu, w, 1, q_len, [0], q_len % 2, split)


# 257 to 512 tokens: down projection in tiles of 128 x 128 over the whole of K with the closing sync point behind it (from 96 tiles on: 25 m-tiles
# of 105 pairs, 17 of 129, none below), O projection in such tiles from 512 workgroups of the skinny kernel on (129 pairs: 25 m-tiles); n-tiles that end
# inside a tile, an odd number of k-tiles
DOWN_129 = Workload(name="129-pairs-51-k-tiles", hidden=4128, n_q_heads=10, n_kv_heads=2, head_dim=32, ffn=3232, n_layers=2, tp=2, dtype=BF16,
                    seed=62, batch=1, q_len=1, ctx=64, mask=(1, 0))
DOWN_105 = Workload(name="105-pairs-51-k-tiles", hidden=3360, n_q_heads=10, n_kv_heads=2, head_dim=32, ffn=3232, n_layers=2, tp=2, dtype=BF16,
                    seed=63, batch=1, q_len=1, ctx=64, mask=(0, 1))


@pytest.mark.parametrize("w", [DOWN_129, DOWN_105], ids=lambda w: w.name)
@pytest.mark.parametrize("q_len,flag,split", [(256, 1, 0), (257, 0, 0), (257, 1, 1), (384, 1, 0), (385, 0, 0), (400, 1, 1), (512, 0, 0), (512, 1, 2)])
def test_bf16_medium_call_in_square_tiles(gpu, w, q_len, flag, split):
    _one_rank_block(gpu, w, 1, q_len, [0], flag, split, bias_std=0.1 * (q_len % 2))


# O projection on either side of 640 workgroups of the skinny kernel (two pairs and four m-tiles each): 160 and 176 pairs at 25 and 32 m-tiles; 512 of
# 256 pairs at 9 and 16, 768 at 17
O_160 = Workload(name="160-pairs", hidden=5120, n_q_heads=10, n_kv_heads=2, head_dim=32, ffn=320, n_layers=1, tp=2, dtype=BF16, seed=68, batch=1,
                 q_len=1, ctx=64, mask=(1,))
O_176 = dataclasses.replace(O_160, name="176-pairs", hidden=5632, seed=69)
O_256 = dataclasses.replace(O_160, name="256-pairs", hidden=8192, seed=70)


@pytest.mark.parametrize("w,q_len", [(O_160, 385), (O_160, 512), (O_176, 385), (O_176, 512), (O_256, 129), (O_256, 256), (O_256, 257)],
                         ids=lambda v: getattr(v, "name", v))
def test_bf16_output_projection_of_medium_call(gpu, w, q_len):
    _one_rank_block(gpu, w, 1, q_len, [0], 1)


# ... and in a model call, where the launch behind it also prepares the next block's first norm: every block against the oracle on the input it had
@pytest.mark.parametrize("w", [DOWN_129, DOWN_105], ids=lambda w: w.name)
def test_bf16_medium_model_call_in_square_tiles(gpu, w):
    import torch
    M, rank = 390, 1
    case = Case(w, gpu, ranks=[rank], positions=[0], max_ctx=416, max_tokens=M, bias_std=0.1)
    X, peers = inputs.hidden_states(w, M), inputs.peer_slots(w, M)
    outs, x = torch.zeros((2, M, w.hidden), dtype=torch.float32, device=gpu), case.to_dev(X)
    B.spd_model_forward_staged(case.dev.ctx, w.mask, rank, case.dev.weights, case.dev.kv, [0], 1, M, x, case.to_dev(peers).reshape(w.tp, M, w.hidden),
                               torch.empty_like(x), case.dev.workspace, layer_out=outs)
    torch.cuda.synchronize()
    for l, flag in enumerate(w.mask):
        want = O.block_single_rank(case.sh, X, case.shards[l][0], case.caches[l][0], [0], 1, M, flag, rank,
                                   peers.reshape(w.tp, M, w.hidden).astype(np.float64))
        X = outs[l].cpu().numpy()
        assert_close(X, want, w, f"block {l}")
    case.close()


# the skinny kernel with two pairs of n-tiles and four m-tiles per workgroup (8 m-tiles and more, pairs in sixteens), against one pair and eight (7 m-tiles;
# 100 pairs): O and down of 96 pairs, 12 and 39 k-tiles, m-tiles that end inside a group of four
SKINNY_96 = Workload(name="96-pairs-39-k-tiles", hidden=3072, n_q_heads=24, n_kv_heads=4, head_dim=32, ffn=2496, n_layers=1, tp=2, dtype=BF16,
                     seed=64, batch=1, q_len=1, ctx=64, mask=(1,))
SKINNY_100 = Workload(name="100-pairs-39-k-tiles", hidden=3200, n_q_heads=24, n_kv_heads=4, head_dim=32, ffn=2496, n_layers=1, tp=2, dtype=BF16,
                      seed=65, batch=1, q_len=1, ctx=64, mask=(1,))


@pytest.mark.parametrize("w", [SKINNY_96, SKINNY_100], ids=lambda w: w.name)
@pytest.mark.parametrize("q_len,flag", [(112, 1), (113, 0), (128, 1), (129, 0), (150, 1), (200, 0), (333, 0), (500, 1), (512, 0)])
def test_bf16_skinny_kernel_of_two_pairs(gpu, w, q_len, flag):
    _one_rank_block(gpu, w, 1, q_len, [0], flag, bias_std=0.1 * (q_len % 2))


# Two workgroups of the prefill attention with one column tile per compute unit: a few registers more and there is one
@pytest.mark.parametrize("head_dim", [32, 64, 96, 128])
def test_bf16_prefill_attention_workgroups(gpu, head_dim):
    assert B.lib().spd_prefill_attention_workgroups(head_dim) >= 2
    assert B.lib().spd_prefill_attention_workgroups(head_dim + 16) == B.SPD_EINVAL


# Decode attention on caches of 64 MB and more in all layers of the context, which are read past the chip's caches: a model call's first block and a block
# call of that context have the same bits as a block call of a context of one layer, whose caches are below that, with the QKV projection whole
# and in slices
@pytest.mark.parametrize("head_dim,kv", [(32, 4), (64, 2), (96, 2), (128, 1)])
@pytest.mark.parametrize("hidden", [256, 2048], ids=["whole", "sliced"])
def test_bf16_decode_of_large_caches(gpu, head_dim, kv, hidden):
    import torch
    w = Workload(name=f"kv-{head_dim}", hidden=hidden, n_q_heads=4 * kv, n_kv_heads=2 * kv, head_dim=head_dim, ffn=128, n_layers=11, tp=2, dtype=BF16,
                 seed=66, batch=12, q_len=1, ctx=1056, mask=(1, 0) * 5 + (1,))
    positions = [1055 - 3 * i for i in range(12)]
    assert 4 * kv * head_dim * sum(positions) < 64 << 20 <= 11 * 4 * kv * head_dim * sum(positions)
    shard = B.DeviceShard(w, [0], gpu, max_ctx=1056, max_tokens=12, max_batch=12)
    torch.manual_seed(66)
    for l in range(w.n_layers):
        shard.load_layer(l, [inputs.layer_shard(w, 0, 0)])
        shard.kv[l].view(torch.bfloat16).normal_()
    x, slots = torch.randn(12, hidden, device=gpu), torch.zeros(2, 12, hidden, device=gpu)
    taps, out = torch.zeros(w.n_layers, 12, hidden, device=gpu), torch.empty_like(x)
    kv0 = shard.kv[0].clone()
    one = B.DeviceShard(dataclasses.replace(w, n_layers=1, mask=(1,)), [0], gpu, max_ctx=1056, max_tokens=12, max_batch=12)
    pos = (B.C.c_int32 * 12)(*positions)
    assert [B.lib().spd_decode_past_caches(c, pos, 12) for c in (one.ctx, shard.ctx)] == [0, 1]
    B.spd_block_forward(one.ctx, 0, 1, 0, shard.weights[0], shard.kv[0], positions, 12, 1, x, slots, out, one.workspace)
    torch.cuda.synchronize()
    appended, want = shard.kv[0].clone(), out.clone()
    shard.kv[0].copy_(kv0)
    B.spd_block_forward(shard.ctx, 0, 1, 0, shard.weights[0], shard.kv[0], positions, 12, 1, x, slots.zero_(), out, shard.workspace)
    torch.cuda.synchronize()
    assert torch.isfinite(want).all() and torch.equal(out, want) and torch.equal(shard.kv[0], appended)
    shard.kv[0].copy_(kv0)
    B.spd_model_forward_staged(shard.ctx, w.mask, 0, shard.weights, shard.kv, positions, 12, 1, x, slots.zero_(), out, shard.workspace, layer_out=taps)
    torch.cuda.synchronize()
    assert torch.equal(taps[0], want) and torch.equal(shard.kv[0], appended)
    one.close()
    shard.close()


# A NaN in the keys of a whole split of the context reaches the output, whichever launch merges the splits: the O projection in one piece or three per
# thread, or one of its own
@pytest.mark.parametrize("kv,batch", [(2, 1), (2, 12), (8, 12)], ids=["one-piece", "three-pieces", "own-launch"])
@pytest.mark.parametrize("first,count", [(0, 512), (256, 256), (700, 1)])
def test_bf16_decode_keeps_nan_scores(gpu, kv, batch, first, count):
    import torch
    w = Workload(name="nan", hidden=3072, n_q_heads=4 * kv, n_kv_heads=2 * kv, head_dim=64, ffn=128, n_layers=1, tp=2, dtype=BF16, seed=71, batch=batch,
                 q_len=1, ctx=1024, mask=(1,))
    shard = B.DeviceShard(w, [0], gpu, max_ctx=1024, max_tokens=batch, max_batch=batch)
    torch.manual_seed(71)
    shard.load_layer(0, [inputs.layer_shard(w, 0, 0)])
    cache = shard.kv[0].view(torch.bfloat16).normal_()
    x, slots, out = torch.randn(batch, w.hidden, device=gpu), torch.zeros(2, batch, w.hidden, device=gpu), torch.empty(batch, w.hidden, device=gpu)
    call = lambda: B.spd_block_forward(shard.ctx, 0, 1, 0, shard.weights[0], shard.kv[0], [1023] * batch, batch, 1, x, slots.zero_(), out, shard.workspace)
    call()
    torch.cuda.synchronize()
    want = out.clone()
    keys = cache[:batch * kv * 1024 * 64].view(batch, kv, 1024 // 16, 16 * 64)       # (16 positions a block, features in eights)
    if count == 1:
        keys[0, kv - 1, first // 16].view(8, 16, 8)[:, first % 16] = float("nan")
    else:
        keys[0, kv - 1, first // 16:(first + count) // 16] = float("nan")
    call()
    torch.cuda.synchronize()
    assert torch.isfinite(want).all() and torch.isnan(out[0]).all() and torch.equal(out[1:], want[1:])
    shard.close()


# the kernel that adds the slices takes 2, 4 or 8 pairs of n-tiles per workgroup, by the number of groups of 8 times m-tiles (lines at 64 and
# 128): gate/up of 66 pairs (9 groups) on either side of both lines, QKV of 7 pairs
FIN_66 = Workload(name="66-and-7-pairs", hidden=3232, n_q_heads=10, n_kv_heads=2, head_dim=32, ffn=2112, n_layers=1, tp=2, dtype=BF16,
                  seed=47, batch=1, q_len=1, ctx=64, mask=(1,))


@pytest.mark.parametrize("q_len", [17, 112, 113, 224, 225])
def test_bf16_slices_added_by_few_and_many_workgroups(gpu, q_len):
    _one_rank_block(gpu, FIN_66, 1, q_len, [0], q_len % 2)


@pytest.mark.parametrize("q_len,flag", [(17, 1), (40, 0), (100, 1)])
def test_bf16_short_call_of_a_wide_model(gpu, q_len, flag):
    """More pairs of n-tiles (520 in the O and down projections) than compute units, and two sync-point epilogues on them."""
    _one_rank_block(gpu, ROWS_65, 1, q_len, [0], flag)


# decode steps whose O projection merges the attention's splits itself (one or up to three quads of features per thread, 512 and 1536 of them; 40 k-tiles)
# and the first beyond: one k-tile
# (waves without any), 9, 32, 40 and 41; groups of 1, 3 and 4 heads; an empty cache, and more than 16 splits
@pytest.mark.parametrize("heads,kv_heads,head_dim,batches", [(2, 2, 32, (1, 16)), (6, 2, 96, (7, 8, 16)), (16, 4, 128, (2, 3, 6, 7)), (80, 80, 32, (1, 2)),
                                                             (82, 82, 32, (1,))], ids=["1-k-tile", "9", "32", "40", "41"])
@pytest.mark.parametrize("flag", [1, 0], ids=["spd", "tp"])
def test_bf16_decode_merge_of_splits(gpu, heads, kv_heads, head_dim, batches, flag):
    w = Workload(name=f"merge-{heads}x{head_dim}", hidden=3072, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=head_dim, ffn=256, n_layers=1,
                 tp=2, dtype=BF16, seed=48, batch=1, q_len=1, ctx=64, mask=(flag,))
    for b in batches:
        _one_rank_block(gpu, w, b, 1, [(i * 211) % 700 for i in range(b)], flag)
    _one_rank_block(gpu, w, 1, 1, [2300], flag)


# Taps leave the launches as they are where the O projection merges the splits (the tapped attention output comes from the merging kernel's launch
# beside it): the same bits with and without taps.  One, two and three quads per thread, and more splits than the first chunk of 16.
@pytest.mark.parametrize("heads,batch,pos", [(2, 3, 700), (8, 4, 500), (8, 6, 900), (8, 1, 3000)])
def test_bf16_tapped_call_is_the_ordinary_call(gpu, heads, batch, pos):
    import torch
    w = Workload(name="tapped", hidden=3072, n_q_heads=heads, n_kv_heads=heads // 2, head_dim=128, ffn=256, n_layers=1, tp=1, dtype=BF16, seed=53,
                 batch=1, q_len=1, ctx=64, mask=(1,))
    for seed in range(4):
        positions = [pos - 97 * ((i + seed) % 5) for i in range(batch)]
        case = Case(w, gpu, ranks=[0], positions=positions, max_ctx=(pos + 32) // 32 * 32, max_tokens=batch)
        X = inputs.hidden_states(w, batch) * (1 + seed)
        got = []
        for tapped in (False, True):
            slots = torch.zeros((1, batch, w.hidden), dtype=torch.float32, device=gpu)
            x = case.to_dev(X)
            if tapped:
                got.append((_block_with_taps(case, 0, 1, 0, x, slots, batch, 1, positions)[0], slots))
            else:
                out = torch.empty_like(x)
                B.spd_block_forward(case.dev.ctx, 0, 1, 0, case.dev.weights[0], case.dev.kv[0], positions, batch, 1, x, slots, out, case.dev.workspace)
                got.append((out, slots))
            torch.cuda.synchronize()
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), seed
        case.close()


# more (sequence, KV head) pairs than a launch takes along one dimension of its grid (65536): the merging kernel's is over heads and sequences
def test_bf16_decode_many_heads_and_sequences(gpu):
    w = Workload(name="1040-heads", hidden=64, n_q_heads=1040, n_kv_heads=1040, head_dim=32, ffn=32, n_layers=1, tp=1, dtype=BF16, seed=57,
                 batch=1, q_len=1, ctx=64, mask=(1,))
    _one_rank_block(gpu, w, 64, 1, [i % 3 for i in range(64)], 1, max_ctx=32, rank=0)


# A call with only the O projection's stage launches what the ordinary call launches, on what that call left: its partial sums come out again
@pytest.mark.parametrize("heads,batch,pos", [(4, 3, 700), (16, 6, 900), (16, 16, 900)])
def test_bf16_o_stage_alone(gpu, heads, batch, pos):
    import torch
    w = Workload(name="o-alone", hidden=3072, n_q_heads=heads, n_kv_heads=heads // 2, head_dim=128, ffn=256, n_layers=1, tp=2, dtype=BF16, seed=54,
                 batch=1, q_len=1, ctx=64, mask=(0,))
    positions = [pos - 97 * (i % 5) for i in range(batch)]
    x = torch.from_numpy(inputs.hidden_states(w, batch)).to(gpu)
    got = []
    for ahat_of in (0, 1):               # another call in between, whose attention output must not be what the O projection reads
        case = Case(w, gpu, ranks=[0], positions=positions, max_ctx=(pos + 32) // 32 * 32, max_tokens=batch)
        peers = case.to_dev(inputs.peer_slots(w, batch)).reshape(w.tp, batch, w.hidden)
        args = lambda xx, sl: (case.dev.ctx, w.mask, 0, case.dev.weights, case.dev.kv, positions, batch, 1, xx, sl, torch.empty_like(xx), case.dev.workspace)
        if ahat_of:
            B.spd_model_forward(*args(x * -2.0 + 1.0, peers.clone()))
        B.spd_model_forward(*args(x, peers.clone()))
        slots = peers.clone()
        B.spd_model_forward_staged(*args(x, slots), stage_mask=1 << 3)
        torch.cuda.synchronize()
        got.append(slots[0])
        case.close()
    assert torch.isfinite(got[0]).all() and float(got[0].abs().max()) > 0
    assert torch.equal(got[0], got[1])


# decode steps whose QKV projection reads the residual stream itself (up to 8 sequences, slices in one round of the chip): waves with one to six of its
# k-tiles (161 in two slices; 64 in two), the first number of sequences beyond; the output in the input's place
QKV_161 = Workload(name="qkv-161-k-tiles", hidden=5152, n_q_heads=20, n_kv_heads=20, head_dim=128, ffn=64, n_layers=1, tp=2, dtype=BF16,
                   seed=50, batch=1, q_len=1, ctx=64, mask=(1,))


@pytest.mark.parametrize("w", [QKV_161, QKV_96], ids=lambda w: w.name)
@pytest.mark.parametrize("flag", [1, 0], ids=["spd", "tp"])
@pytest.mark.parametrize("batch", [1, 5, 8, 9])
def test_bf16_decode_first_norm_in_qkv(gpu, w, flag, batch):
    import torch
    positions = [(11 * i) % 61 for i in range(batch)]
    _one_rank_block(gpu, w, batch, 1, positions, flag, max_ctx=64)
    case = Case(w, gpu, ranks=range(w.tp), positions=positions, max_ctx=64, max_tokens=batch)
    X = inputs.hidden_states(w, batch)
    x, slots = case.to_dev(X), torch.zeros((w.tp, batch, w.hidden), dtype=torch.float32, device=gpu)
    B.spd_block_forward(case.dev.ctx, 0, flag, B.SPD_ALL_RANKS, case.dev.weights[0], case.dev.kv[0], positions, batch, 1, x, slots, x,
                        case.dev.workspace)
    torch.cuda.synchronize()
    want, _ = O.block_all_ranks(case.sh, X, case.shards[0], case.caches[0], positions, batch, 1, flag, {})
    assert_close(x.cpu().numpy(), want, w, "block output, all ranks")
    case.close()


# A timer on a stage, or the blocks' outputs asked for, leave a call's launches as they are: the same bits
@pytest.mark.parametrize("batch", [1, 5, 8, 9])
def test_bf16_timed_call_is_the_ordinary_call(gpu, batch):
    import torch
    w = Workload(name="timed", hidden=2048, n_q_heads=16, n_kv_heads=16, head_dim=128, ffn=256, n_layers=2, tp=2, dtype=BF16, seed=52, batch=1,
                 q_len=1, ctx=64, mask=(1, 0))
    positions = [(13 * i + 9) % 61 for i in range(batch)]
    case = Case(w, gpu, ranks=[1], positions=positions, max_ctx=64, max_tokens=batch)
    x, peers = case.to_dev(inputs.hidden_states(w, batch)), case.to_dev(inputs.peer_slots(w, batch)).reshape(w.tp, batch, w.hidden)
    got = []
    for stage in [None, "layer_out"] + list(range(B.SPD_ALL_STAGES.bit_length())):
        timer = B.spd_stage_timer_create(stage, 8) if isinstance(stage, int) else None
        slots, out = peers.clone(), torch.empty_like(x)
        kw = {} if stage is None else {"timer": timer} if timer else {"layer_out": torch.empty((2, batch, w.hidden), device=gpu)}
        f = B.spd_model_forward if stage is None else B.spd_model_forward_staged
        f(case.dev.ctx, w.mask, 1, case.dev.weights, case.dev.kv, positions, batch, 1, x, slots, out, case.dev.workspace, **kw)
        torch.cuda.synchronize()
        if timer:
            B.spd_stage_timer_destroy(timer)
        got.append((out, slots))
        assert torch.equal(out, got[0][0]) and torch.equal(slots, got[0][1]), stage
    case.close()


# The first norm's product x * gain is rounded to fp16 once, in the QKV projection (up to 8 sequences) as in the preparation's launch: every second
# element is (1 + 2^-12)^2, a little above a tie of fp16, the others are 1 and counted with the other sign.  The values are then
# the sum of 1024 times 2^-10; of products rounded to 32 bits first, which are ties and become 1, they are 0.
@pytest.mark.parametrize("batch", [1, 8, 9])
def test_bf16_decode_first_norm_rounds_once(gpu, batch):
    import torch
    w = Workload(name="round-once", hidden=2048, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=64, n_layers=1, tp=1, dtype=BF16, seed=51,
                 batch=1, q_len=1, ctx=32, mask=(1,))
    shard = B.DeviceShard(w, [0], gpu, max_ctx=32, max_tokens=batch, max_batch=batch)
    s = inputs.layer_shard(w, 0, 0)
    s["g1"] = np.ones(w.hidden, np.float32)
    s["g1"][::2] += 2.0 ** -12
    s["wv"] = np.full_like(s["wv"], 1.0)
    s["wv"][1::2] = -1.0
    shard.load_layer(0, [s])
    x = torch.from_numpy(np.tile(s["g1"], (batch, 1))).to(gpu)
    slots, out = torch.zeros((1, batch, w.hidden), dtype=torch.float32, device=gpu), torch.empty_like(x)
    B.spd_block_forward(shard.ctx, 0, 1, 0, shard.weights[0], shard.kv[0], [0] * batch, batch, 1, x, slots, out, shard.workspace)
    torch.cuda.synchronize()
    _, v = B.spd_kv_unpack(shard.ctx, shard.kv[0].cpu().numpy(), batch, 1, w.kv_per_rank, w.head_dim)
    # 2^-8 relative: the value's rounding to bf16; the norm's factor differs from 1 by 3e-4
    assert np.all(np.abs(np.asarray(v) - 1.0) <= 2.0 ** -8 + 1e-3), np.asarray(v).ravel()[:4]
    shard.close()


# decode QKV projections of 192 pairs and more, which the attention kernel does not add up: one launch up to 160 k-tiles
QKV_192 = Workload(name="qkv-192-pairs", hidden=5120, n_q_heads=32, n_kv_heads=32, head_dim=128, ffn=256, n_layers=1, tp=2, dtype=BF16,
                   seed=40, batch=1, q_len=1, ctx=64, mask=(1,))
QKV_192_LONG = Workload(name="qkv-192-pairs-long", hidden=5152, n_q_heads=32, n_kv_heads=32, head_dim=128, ffn=256, n_layers=1, tp=2,
                        dtype=BF16, seed=41, batch=1, q_len=1, ctx=64, mask=(1,))


@pytest.mark.parametrize("w", [QKV_192, QKV_192_LONG], ids=lambda w: w.name)
@pytest.mark.parametrize("batch", [16, 17, 33, 64])
def test_bf16_decode_qkv_of_a_wide_shard(gpu, w, batch):
    _one_rank_block(gpu, w, batch, 1, [(7 * i) % 61 for i in range(batch)], batch % 2, max_ctx=64)


# a kept attention sync point of 129 .. 512 tokens: in the O projection's epilogue up to 512 workgroups (130 pairs x groups of 128
# tokens: 390 up to 384 tokens, 520 beyond) and eight k-tiles per slot, a kernel of its own from there; with bias and with paired
# activations
SYNC_130 = Workload(name="sync-130-pairs", hidden=4160, n_q_heads=8, n_kv_heads=8, head_dim=64, ffn=256, n_layers=1, tp=8, dtype=BF16,
                    seed=43, batch=1, q_len=1, ctx=64, mask=(0,))


SYNC_16_KT = Workload(name="sync-16-k-tiles", hidden=512, n_q_heads=16, n_kv_heads=16, head_dim=64, ffn=256, n_layers=1, tp=2, dtype=BF16,
                      seed=46, batch=1, q_len=1, ctx=64, mask=(0,))
SYNC_18_KT = Workload(name="sync-18-k-tiles", hidden=512, n_q_heads=18, n_kv_heads=18, head_dim=64, ffn=256, n_layers=1, tp=2, dtype=BF16,
                      seed=47, batch=1, q_len=1, ctx=64, mask=(0,))


@pytest.mark.parametrize("w", [SYNC_16_KT, SYNC_18_KT], ids=lambda w: w.name)
@pytest.mark.parametrize("q_len", [128, 300])
def test_bf16_kept_sync_point_of_two_ranks(gpu, w, q_len):
    _one_rank_block(gpu, w, 1, q_len, [0], 0)


@pytest.mark.parametrize("bias_std,split", [(0.0, B.SPD_SPLIT_AUTO), (1.0, B.SPD_SPLIT_AUTO), (0.0, B.SPD_SPLIT_ALWAYS)],
                         ids=["plain", "bias", "all-split"])
@pytest.mark.parametrize("q_len", [128, 129, 300, 384, 385, 512])
def test_bf16_kept_sync_point_of_a_medium_call(gpu, q_len, bias_std, split):
    _one_rank_block(gpu, SYNC_130, 1, q_len, [0], 0, split, bias_std=bias_std)


# the weight-streaming kernel's ring of k-tiles: shares of a wave shorter than the ring, of one and of several turns, with every number of k-tiles
# left over (down: 33, 81, 100 and 145 k-tiles over 16 waves in one launch, 1 in a wave each; gate/up: 192, in slices)
@pytest.mark.parametrize("k_tiles", [1, 33, 81, 100, 145])
@pytest.mark.parametrize("split", [B.SPD_SPLIT_AUTO, B.SPD_SPLIT_ALWAYS], ids=["default", "all-split"])
@pytest.mark.parametrize("flag", [1, 0], ids=["spd", "tp"])
def test_bf16_decode_contraction_lengths(gpu, k_tiles, split, flag):
    w = Workload(name=f"down-{k_tiles}-k-tiles", hidden=6144, n_q_heads=2, n_kv_heads=2, head_dim=32, ffn=64 * k_tiles, n_layers=1, tp=2,
                 dtype=BF16, seed=48, batch=1, q_len=1, ctx=64, mask=(flag,))
    _one_rank_block(gpu, w, 5, 1, [3, 0, 40, 17, 31], flag, split)


# sync points in epilogues that ask for the first eight slots ahead of the contraction: fewer slots, as many, more, and an own slot beyond them
@pytest.mark.parametrize("tp,rank", [(1, 0), (2, 0), (8, 7), (9, 8), (9, 3), (16, 11)])
@pytest.mark.parametrize("batch,flag", [(3, 0), (16, 1), (24, 0), (48, 1), (64, 0)])
def test_bf16_sync_point_of_several_ranks(gpu, tp, rank, batch, flag):
    w = Workload(name=f"{tp}-ranks", hidden=512, n_q_heads=2 * tp, n_kv_heads=tp, head_dim=32, ffn=96 * tp, n_layers=1, tp=tp,
                 dtype=BF16, seed=49, batch=1, q_len=1, ctx=64, mask=(flag,))
    _one_rank_block(gpu, w, batch, 1, [(7 * i) % 61 for i in range(batch)], flag, max_ctx=64, bias_std=batch % 3 * 0.5, rank=rank)


@pytest.mark.parametrize("tp,rank", [(1, 0), (8, 7), (9, 8), (16, 11)])
@pytest.mark.parametrize("q_len,flag", [(100, 0), (128, 1), (200, 0)])
def test_bf16_sync_point_of_several_ranks_short_prompt(gpu, tp, rank, q_len, flag):
    w = Workload(name=f"{tp}-ranks", hidden=512, n_q_heads=2 * tp, n_kv_heads=tp, head_dim=32, ffn=96 * tp, n_layers=1, tp=tp,
                 dtype=BF16, seed=49, batch=1, q_len=1, ctx=64, mask=(flag,))
    _one_rank_block(gpu, w, 1, q_len, [0], flag, rank=rank)


# fp32 path at the edges of its small-product kernel (at most 64 rows and 1024 contraction elements, rotation inside it when the
# head size divides its 64 columns): odd widths, a head size that does not divide 64, one row, a full and a
# started 8-row tile, the last size inside the range and the first beyond it in rows and in K
F32_ODD = Workload(name="f32-odd", hidden=131, n_q_heads=6, n_kv_heads=2, head_dim=10, ffn=154, n_layers=1, tp=2, dtype=F32,
                   seed=41, batch=1, q_len=1, ctx=96, mask=(1,))
F32_HEADS = Workload(name="f32-d32", hidden=1024, n_q_heads=4, n_kv_heads=4, head_dim=32, ffn=2050, n_layers=1, tp=2, dtype=F32,
                     seed=42, batch=1, q_len=1, ctx=96, mask=(1,))
F32_WIDE = Workload(name="f32-k1025", hidden=1025, n_q_heads=2, n_kv_heads=2, head_dim=64, ffn=64, n_layers=1, tp=2, dtype=F32,
                    seed=43, batch=1, q_len=1, ctx=96, mask=(1,))


@pytest.mark.parametrize("w", [F32_ODD, F32_HEADS, F32_WIDE], ids=lambda w: w.name)
@pytest.mark.parametrize("flag", [1, 0], ids=["spd", "tp"])
@pytest.mark.parametrize("batch,q_len,positions", [(1, 1, [0]), (2, 4, [0, 13]), (3, 3, [5, 0, 30]), (1, 64, [7]), (1, 65, [0])],
                         ids=["1", "8", "9", "64", "65"])
def test_fp32_small_products(gpu, w, flag, batch, q_len, positions):
    import torch
    M = batch * q_len
    case = Case(w, gpu, ranks=range(w.tp), positions=positions, max_ctx=96, max_tokens=M)
    X = inputs.hidden_states(w, M)
    slots = torch.zeros((w.tp, M, w.hidden), dtype=torch.float32, device=gpu)
    say(f"fp32 small products: {w.name} {M} tokens flag={flag}")
    out = torch.empty((M, w.hidden), dtype=torch.float32, device=gpu)
    B.spd_block_forward(case.dev.ctx, 0, flag, B.SPD_ALL_RANKS, case.dev.weights[0], case.dev.kv[0], positions, batch, q_len,
                        case.to_dev(X), slots, out, case.dev.workspace)
    torch.cuda.synchronize()
    want, _ = O.block_all_ranks(case.sh, X, case.shards[0], case.caches[0], positions, batch, q_len, flag, {})
    err = assert_close(out.cpu().numpy(), want, w, "block output", scale=0.02)      # 2e-5: some 20 roundings of fp32 over K <= 2050
    say(f"  block output max err {err:.2e}")
    case.close()


# Small fp32 calls run the ranks side by side, one to eight rows of up to 256, 512 or 1024 elements per workgroup, and perform the sums over
# the ranks but the last mostly in the launch that reads them: every block against the oracle on the input it had (sums over at most 768 elements in 32
# bits: 1e-5 of the largest), and the same bits whether the blocks' outputs, a stage's time or nothing is asked for.
@pytest.mark.parametrize("hidden,ffn", [(96, 1560), (257, 768), (768, 90)], ids=["k520", "k257", "k768"])
@pytest.mark.parametrize("rank", [None, 1], ids=["all-ranks", "one-rank"])
@pytest.mark.parametrize("batch,q_len,positions", [(1, 1, [31]), (5, 1, [0, 9, 30, 2, 31]), (1, 33, [3]), (2, 32, [0, 32])], ids=["1", "5", "33", "64"])
def test_fp32_ranks_side_by_side(gpu, hidden, ffn, rank, batch, q_len, positions):
    import torch
    w = Workload(name=f"f32-side-{hidden}-{ffn}", hidden=hidden, n_q_heads=6, n_kv_heads=3, head_dim=32, ffn=ffn, n_layers=4, tp=3, dtype=F32,
                 seed=46, batch=1, q_len=1, ctx=64, mask=(1, 0, 0, 1))
    M = batch * q_len
    X, peers = inputs.hidden_states(w, M), inputs.peer_slots(w, M)
    say(f"fp32 side by side: {w.name} rank={rank} {M} tokens")
    got = []
    for how in ("plain", "layer_out", "timer"):
        case = Case(w, gpu, ranks=range(w.tp) if rank is None else [rank], positions=positions, max_ctx=64, max_tokens=M, bias_std=1.0)
        slots = case.to_dev(peers).reshape(w.tp, M, w.hidden)
        x = case.to_dev(X)                       # the output takes the input's place
        outs = torch.zeros((w.n_layers, M, w.hidden), dtype=torch.float32, device=gpu)
        timer = B.spd_stage_timer_create(4, 16) if how == "timer" else None
        args = (case.dev.ctx, w.mask, case.dev.rank_arg(), case.dev.weights, case.dev.kv, positions, batch, q_len, x, slots, x, case.dev.workspace)
        if how == "plain":
            syncs = B.spd_model_forward(*args)
        else:
            syncs = B.spd_model_forward_staged(*args, **({"timer": timer} if timer else {"layer_out": outs}))
        torch.cuda.synchronize()
        assert syncs == 6
        if timer:
            assert B.spd_stage_timer_read(timer)[0] == w.n_layers
            B.spd_stage_timer_destroy(timer)
        got.append([x, slots] + [k.view(torch.float32) for k in case.dev.kv])
        for a, b in zip(got[0], got[-1]):
            assert torch.equal(a, b), how
        if how == "layer_out":
            outs, xb = outs.cpu().numpy().astype(np.float64), X
            assert np.array_equal(outs[-1], x.cpu().numpy())
            for l, flag in enumerate(w.mask):
                if rank is None:
                    want, _ = O.block_all_ranks(case.sh, xb, case.shards[l], case.caches[l], positions, batch, q_len, flag, {})
                else:
                    want = O.block_single_rank(case.sh, xb, case.shards[l][0], case.caches[l][0], positions, batch, q_len, flag, rank,
                                               peers.reshape(w.tp, M, w.hidden).astype(np.float64))
                assert np.max(np.abs(outs[l] - want)) <= 1e-5 * np.max(np.abs(want)), l
                xb = outs[l].astype(np.float32)
        case.close()


# The norm's factor of a call of one token, whose row 16 waves load: one element of 2^12 in the first part of the row and a 1 in each of the others, which
# a sum of the parts one after the other loses against 2^24.  The factor would be off by 15 / 2^25 = 4.5e-7; roundings leave 2e-7 at most
# (the mean, the root's argument by half, the root, its inverse, two products: half a unit in the last place each).
def test_fp32_norm_of_one_token(gpu):
    import torch
    w = Workload(name="f32-norm", hidden=256, n_q_heads=2, n_kv_heads=2, head_dim=32, ffn=64, n_layers=1, tp=1, dtype=F32, seed=58, batch=1,
                 q_len=1, ctx=32, mask=(1,))
    shard = B.DeviceShard(w, [0], gpu, max_ctx=32, max_tokens=1, max_batch=1)
    s = inputs.layer_shard(w, 0, 0)
    s["g1"] = np.ones(w.hidden, np.float32)
    s["wv"] = np.zeros_like(s["wv"])
    s["wv"][0] = 1.0
    shard.load_layer(0, [s])
    x = np.zeros((1, w.hidden), np.float32)
    x[0, ::16] = 1.0
    x[0, 0] = 4096.0
    xd = torch.from_numpy(x).to(gpu)
    slots, out = torch.zeros((1, 1, w.hidden), dtype=torch.float32, device=gpu), torch.empty_like(xd)
    B.spd_block_forward(shard.ctx, 0, 1, 0, shard.weights[0], shard.kv[0], [0], 1, 1, xd, slots, out, shard.workspace)
    torch.cuda.synchronize()
    _, v = B.spd_kv_unpack(shard.ctx, shard.kv[0].cpu().numpy(), 1, 1, w.kv_per_rank, w.head_dim)
    want = 4096.0 / np.sqrt(np.mean(x.astype(np.float64) ** 2) + w.rms_eps)
    assert np.max(np.abs(np.asarray(v, np.float64) / want - 1.0)) <= 2.5e-7
    shard.close()


# Where a sum over the ranks is done: in the launch of the product that reads it up to 4 MiB of slots read (16 MiB with up to 32 slots), by a launch of
# its own beyond (counted by a timer on its stage).  Two layers, the kept sync point and the end of the first block on either side of the lines.
@pytest.mark.parametrize("tp,rank,M,ffn,launches", [(34, 1, 30, 64, 1), (34, 1, 40, 64, 2), (34, 1, 64, 64, 3), (32, 1, 64, 256, 1), (32, 1, 64, 320, 2),
                                                    (8, None, 64, 128, 1), (8, None, 64, 192, 2)])
def test_fp32_sums_over_many_ranks(gpu, tp, rank, M, ffn, launches):
    import torch
    w = Workload(name=f"f32-sums-{tp}", hidden=512, n_q_heads=tp, n_kv_heads=tp, head_dim=32, ffn=ffn * tp, n_layers=2, tp=tp, dtype=F32, seed=55,
                 batch=1, q_len=1, ctx=64, mask=(0, 1))
    X, peers = inputs.hidden_states(w, M), inputs.peer_slots(w, M)
    timer = B.spd_stage_timer_create(0, 16)
    for t in (timer, None):
        case = Case(w, gpu, ranks=range(tp) if rank is None else [rank], positions=[0], max_ctx=64, max_tokens=M, bias_std=1.0)
        slots, out = case.to_dev(peers).reshape(tp, M, w.hidden), torch.empty((M, w.hidden), device=gpu)
        B.spd_model_forward_staged(case.dev.ctx, w.mask, case.dev.rank_arg(), case.dev.weights, case.dev.kv, [0], 1, M, case.to_dev(X), slots, out,
                                   case.dev.workspace, timer=t)
        torch.cuda.synchronize()
        if t:
            assert B.spd_stage_timer_read(timer)[0] == launches
        if rank is None:
            want, _ = O.model_all_ranks(case.sh, X, case.shards, case.caches, [0], 1, M, w.mask)
        else:
            p64, want = peers.reshape(tp, M, w.hidden).astype(np.float64), X
            for l, flag in enumerate(w.mask):
                want = O.block_single_rank(case.sh, want, case.shards[l][0], case.caches[l][0], [0], 1, M, flag, rank, p64)
        # (two layers in 32 bits, sums over 512 elements)
        assert np.max(np.abs(out.cpu().numpy() - want)) <= 2e-5 * np.max(np.abs(want))
        case.close()
    B.spd_stage_timer_destroy(timer)


# A block call with taps takes the ordinary call's launches too: the same bits, and the taps against the oracle
@pytest.mark.parametrize("flag", [1, 0], ids=["spd", "tp"])
@pytest.mark.parametrize("q_len", [1, 33])
def test_fp32_tapped_call_is_the_ordinary_call(gpu, flag, q_len):
    import torch
    w = workloads.TOY
    case = Case(w, gpu, ranks=range(w.tp), positions=[5], max_ctx=64, max_tokens=q_len)
    x = case.to_dev(inputs.hidden_states(w, q_len))
    slots = torch.zeros((w.tp, q_len, w.hidden), dtype=torch.float32, device=gpu)
    slots2, out2 = slots.clone(), torch.empty_like(x)
    out, _ = _block_with_taps(case, 0, flag, B.SPD_ALL_RANKS, x, slots, 1, q_len, [5])
    B.spd_block_forward(case.dev.ctx, 0, flag, B.SPD_ALL_RANKS, case.dev.weights[0], case.dev.kv[0], [5], 1, q_len, x, slots2, out2,
                        case.dev.workspace)
    torch.cuda.synchronize()
    assert torch.equal(out, out2) and torch.equal(slots, slots2)
    case.close()


# The O projection of a small call does the attention itself for up to 16 (row, head) items a workgroup (1, 2, 4 or 8 rows) and 16 keys per wave of an
# item, a launch of its own beyond (counted by a timer on its stage): against the oracle, and against that launch, which a call of one stage
# after the other takes (sums over at most 256 keys in 32 bits: 1e-5 of the largest).
@pytest.mark.parametrize("hidden,tp,q,kv,d,batch,q_len,positions,fused", [
    (64, 1, 16, 16, 32, 1, 1, [15], True), (64, 1, 16, 4, 32, 1, 1, [16], False), (64, 1, 17, 17, 32, 1, 1, [0], False),
    (96, 1, 3, 1, 64, 2, 1, [79, 3], True), (96, 1, 3, 3, 64, 2, 1, [3, 80], False), (64, 2, 1, 1, 64, 1, 1, [255], True),
    (64, 1, 1, 1, 64, 1, 1, [256], False), (64, 1, 1, 1, 16, 1, 1, [3], False), (1024, 1, 2, 2, 64, 1, 32, [32], True),
    (1024, 1, 2, 1, 32, 4, 16, [0, 3, 1, 16], True), (1024, 1, 1, 1, 64, 3, 11, [0, 53, 7], True), (1024, 2, 2, 2, 64, 4, 16, [0] * 4, True)])
def test_fp32_attention_in_the_output_projection(gpu, hidden, tp, q, kv, d, batch, q_len, positions, fused):
    import torch
    w = Workload(name=f"f32-att-{q}x{d}", hidden=hidden, n_q_heads=q * tp, n_kv_heads=kv * tp, head_dim=d, ffn=64 * tp, n_layers=1, tp=tp, dtype=F32,
                 seed=61, batch=1, q_len=1, ctx=288, mask=(0,))
    M, S = batch * q_len, B.STAGES
    case = Case(w, gpu, ranks=range(tp), positions=positions, max_ctx=288, max_tokens=M)
    X = inputs.hidden_states(w, M)
    x, got = case.to_dev(X), []
    timer = B.spd_stage_timer_create(S["attn"], 4)
    for masks in ([(1 << S["qkv"]) | (1 << S["attn"]) | (1 << S["o"])], [1 << S["qkv"], 1 << S["attn"], 1 << S["o"]]):
        slots, out = torch.zeros((tp, M, hidden), dtype=torch.float32, device=gpu), torch.empty_like(x)
        for mask in masks:
            B.spd_model_forward_staged(case.dev.ctx, w.mask, B.SPD_ALL_RANKS, case.dev.weights, case.dev.kv, positions, batch, q_len, x, slots, out,
                                       case.dev.workspace, stage_mask=mask, timer=timer)
        torch.cuda.synchronize()
        assert B.spd_stage_timer_read(timer)[0] == (0 if fused and not got else 1)
        got.append(slots.cpu().numpy())
    B.spd_stage_timer_destroy(timer)
    assert np.max(np.abs(got[0] - got[1])) <= 1e-5 * np.max(np.abs(got[1]))
    assert fused or np.array_equal(got[0], got[1])
    B.spd_block_forward(case.dev.ctx, 0, 0, B.SPD_ALL_RANKS, case.dev.weights[0], case.dev.kv[0], positions, batch, q_len, x, slots, out,
                        case.dev.workspace)
    torch.cuda.synchronize()
    want, _ = O.block_all_ranks(case.sh, X, case.shards[0], case.caches[0], positions, batch, q_len, 0, {})
    assert np.max(np.abs(out.cpu().numpy() - want)) <= 1e-5 * np.max(np.abs(want))
    case.close()


# ... and keys without a score (NaN, inf - inf) make their sequence's row NaN, as in the attention's own launch, and leave the other row alone: all the keys
# that a wave has (the newest one, which is alone in its wave at 9 and 17; an aligned block of eight), all of the sequence's, or one of a wave's eight
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("first,count", [(-1, 1), (0, 8), (0, 40), (3, 1)], ids=["newest", "block", "all", "one"])
@pytest.mark.parametrize("n_keys", [9, 17, 40])
def test_fp32_attention_in_the_output_projection_keeps_nan(gpu, n_keys, first, count, value):
    import torch
    w = Workload(name="f32-att-nan", hidden=64, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=64, n_layers=1, tp=1, dtype=F32, seed=67, batch=1, q_len=1,
                 ctx=64, mask=(0,))
    positions, S = [n_keys - 1, 20], B.STAGES
    first = n_keys + first if first < 0 else first
    case = Case(w, gpu, ranks=[0], positions=positions, max_ctx=64, max_tokens=2)
    x, out, got = case.to_dev(inputs.hidden_states(w, 2)), torch.empty((2, 64), dtype=torch.float32, device=gpu), []
    timer = B.spd_stage_timer_create(S["attn"], 4)

    def call(slots, mask):
        B.spd_model_forward_staged(case.dev.ctx, w.mask, 0, case.dev.weights, case.dev.kv, positions, 2, 1, x, slots, out, case.dev.workspace,
                                   stage_mask=mask, timer=timer)

    for masks in ([(1 << S["attn"]) | (1 << S["o"])], [1 << S["attn"], 1 << S["o"]]):
        slots = torch.zeros((1, 2, 64), dtype=torch.float32, device=gpu)
        call(slots, 1 << S["qkv"])
        # (infinities of both signs, so that the score has no value in whatever order it is summed)
        case.dev.kv[0].view(torch.float32)[:64 * 64].view(64, 64)[first:min(first + count, n_keys)] = torch.tensor([value, -value] * 32, device=gpu)
        for mask in masks:
            call(slots, mask)
        torch.cuda.synchronize()
        assert B.spd_stage_timer_read(timer)[0] == len(got)      # the fused launch first
        got.append(slots[0].cpu().numpy())
    B.spd_stage_timer_destroy(timer)
    for g in got:
        assert np.isnan(g[0]).all() and np.isfinite(g[1]).all()
    assert np.max(np.abs(got[0][1] - got[1][1])) <= 1e-5 * np.max(np.abs(got[1][1]))
    case.close()


# fp32 attention where a thread takes a second key (256 keys and more), the waves' shares end unevenly and the output needs a
# second and a fourth pass of 64 features
@pytest.mark.parametrize("head_dim", [2, 64, 66, 128, 256])
@pytest.mark.parametrize("batch,q_len,positions", [(3, 1, [254, 255, 256]), (2, 1, [257, 1000]), (1, 40, [230])], ids=["256", "1001", "chunk"])
def test_fp32_attention_edges(gpu, head_dim, batch, q_len, positions):
    w = Workload(name=f"f32-attn-d{head_dim}", hidden=64, n_q_heads=4, n_kv_heads=2, head_dim=head_dim, ffn=64, n_layers=1, tp=2, dtype=F32,
                 seed=45, batch=1, q_len=1, ctx=64, mask=(1,))
    # 2e-5 of the largest output: some 20 roundings of fp32 over at most 1001 keys
    _one_rank_block(gpu, w, batch, q_len, positions, 1, bound_scale=0.02)


# ... and at its widest product: 2048 workgroups of 64 columns x 8 rows, and one column more
@pytest.mark.parametrize("ffn", [16384, 16385])
@pytest.mark.parametrize("q_len", [57, 64])
def test_fp32_small_products_width(gpu, ffn, q_len):
    w = Workload(name=f"f32-wide-{ffn}", hidden=64, n_q_heads=4, n_kv_heads=4, head_dim=32, ffn=2 * ffn, n_layers=1, tp=2, dtype=F32, seed=44,
                 batch=1, q_len=1, ctx=64, mask=(1,))
    # (the bound of the fp32 path with 0.1: 1e-4, the down projection sums 16384 products in fp32 one after the other)
    _one_rank_block(gpu, w, 1, q_len, [0], 1, bound_scale=0.1)


# ------------------------------------------------------------------------------------------------
# block with bias in the output projection (Sec. 4.1.2): both paths, both block kinds
# ------------------------------------------------------------------------------------------------
TOY_BIAS = Workload(name="toy-f32-bias", hidden=128, n_q_heads=4, n_kv_heads=2, head_dim=32, ffn=344, n_layers=3, tp=2,
                    dtype=F32, seed=15, batch=2, q_len=1, ctx=32, mask=(1, 0, 1))
SMALL_BIAS = Workload(name="small-bf16-bias", hidden=256, n_q_heads=8, n_kv_heads=4, head_dim=64, ffn=832, n_layers=3,
                      tp=4, dtype=BF16, seed=16, batch=3, q_len=1, ctx=64, mask=(1, 0, 1))


SMALL_BIAS8 = Workload(name="small-bf16-bias-tp8", hidden=256, n_q_heads=16, n_kv_heads=8, head_dim=32, ffn=1024, n_layers=3,
                       tp=8, dtype=BF16, seed=17, batch=3, q_len=1, ctx=64, mask=(1, 0, 1))


@pytest.mark.parametrize("w", [TOY_BIAS, SMALL_BIAS, SMALL_BIAS8], ids=lambda w: w.name)
@pytest.mark.parametrize("batch,q_len,positions",
                         [(3, 1, [0, 9, 30]), (2, 10, [0, 4]), (2, 40, [0, 8]), (3, 181, [0, 3, 0]), (2, 1030, [0, 8])],
                         ids=["decode", "chunk20", "chunk80", "chunk543", "chunk2060"])
@pytest.mark.parametrize("mode", ["all-ranks", "one-rank"])
def test_block_with_bias(gpu, w, batch, q_len, positions, mode):
    """Three blocks (SPD, TP, SPD) with a bias of the size of the activations on the output projection:
    model forward against the oracle, with every rank emulated and from one rank's point of view (whose bf16 call
    of 2 x 1030 tokens runs as two chains, the bias joining the rank-sums of their preparation kernel: four slots in
    the 4-way shard, eight in the 8-way one)."""
    import torch
    M = batch * q_len
    ranks = list(range(w.tp)) if mode == "all-ranks" else [1]
    case = Case(w, gpu, ranks=ranks, positions=positions, max_ctx=max(64, (max(positions) + q_len + 31) // 32 * 32), max_tokens=max(48, M),
                bias_std=1.0)
    X = inputs.hidden_states(w, M)
    say(f"case {w.name} {mode} batch={batch} q_len={q_len}")
    peers = inputs.peer_slots(w, M) if mode == "one-rank" else np.zeros((w.tp, M, w.hidden), np.float32)
    slots = case.to_dev(peers).reshape(w.tp, M, w.hidden)
    out = torch.empty((M, w.hidden), dtype=torch.float32, device=gpu)
    taps = torch.zeros((w.n_layers, M, w.hidden), dtype=torch.float32, device=gpu)
    syncs = B.spd_model_forward_staged(case.dev.ctx, w.mask, case.dev.rank_arg(), case.dev.weights, case.dev.kv,
                                       positions, batch, q_len, case.to_dev(X), slots, out, case.dev.workspace,
                                       layer_out=taps)
    torch.cuda.synchronize()
    assert syncs == 4
    got = taps.cpu().numpy()
    assert np.array_equal(got[-1], out.cpu().numpy())
    # block by block, the oracle's block fed the same input as the library's: the bound as it stands
    worst = 0.0
    o_slots = peers.astype(np.float64)
    for l in range(w.n_layers):
        x_in = X if l == 0 else got[l - 1]
        if mode == "all-ranks":
            want, _ = O.block_all_ranks(case.sh, x_in, case.shards[l], case.caches[l], positions, batch, q_len, w.mask[l])
        else:
            want = O.block_single_rank(case.sh, x_in, case.shards[l][0], case.caches[l][0], positions, batch, q_len,
                                       w.mask[l], 1, o_slots)
        worst = max(worst, assert_close(got[l], want, w, f"{w.name} {mode} block {l}"))
    say(f"  worst block max err {worst:.2e}")
    case.close()


# ------------------------------------------------------------------------------------------------
# bf16 path, one rank of eight with peer slots as inputs, several layers, mixed mask
# ------------------------------------------------------------------------------------------------
MID = Workload(name="mid-bf16", hidden=1024, n_q_heads=32, n_kv_heads=8, head_dim=128, ffn=11008, n_layers=4,
               tp=8, dtype=BF16, seed=13, batch=5, q_len=1, ctx=256, mask=(1, 0, 1, 1))


@pytest.mark.parametrize("batch,q_len,positions", [(5, 1, [255, 100, 0, 31, 64]), (2, 24, [0, 100])],
                         ids=["decode", "chunk"])
def test_bf16_single_rank_model(gpu, batch, q_len, positions):
    import torch
    w, rank = MID, 3
    M = batch * q_len
    case = Case(w, gpu, ranks=[rank], positions=positions, max_ctx=256, max_tokens=48)
    X = inputs.hidden_states(w, M)
    peers = inputs.peer_slots(w, M)
    # per layer: oracle fed the GPU's layer input
    x = case.to_dev(X)
    slots = case.to_dev(peers)
    worst = 0.0
    for l in range(w.n_layers):
        x_host = x.cpu().numpy()
        out = torch.empty_like(x)
        B.spd_block_forward(case.dev.ctx, l, w.mask[l], rank, case.dev.weights[l], case.dev.kv[l], positions, batch,
                            q_len, x, slots, out, case.dev.workspace)
        torch.cuda.synchronize()
        o_slots = peers.astype(np.float64)
        want = O.block_single_rank(case.sh, x_host, case.shards[l][0], case.caches[l][0], positions, batch, q_len,
                                   w.mask[l], rank, o_slots)
        worst = max(worst, assert_close(out.cpu().numpy(), want, w, f"mid layer {l}"))
        # the slot this rank wrote must be what the oracle's rank contributes to the last sync point
        assert_close(slots[rank].cpu().numpy(), o_slots[rank], w, f"mid slot layer {l}")
        # peers untouched, bit for bit
        for i in range(w.tp):
            if i != rank:
                assert np.array_equal(slots[i].cpu().numpy(), peers[i])
        x = out
    say(f"mid {q_len=}: worst per-layer err {worst:.2e}")
    chain = x.cpu().numpy()

    # end to end through spd_model_forward on fresh caches.  It fuses each block's closing rank-sum
    # into the down projection, so the norm statistics are added in another (fixed) order than in
    # the block-by-block chain: equal up to rounding, not bit for bit
    case2 = Case(w, gpu, ranks=[rank], positions=positions, max_ctx=256, max_tokens=48)
    slots2 = case2.to_dev(peers)
    out2 = torch.empty((M, w.hidden), dtype=torch.float32, device=gpu)
    syncs = B.spd_model_forward(case2.dev.ctx, w.mask, rank, case2.dev.weights, case2.dev.kv, positions, batch, q_len,
                                case2.to_dev(X), slots2, out2, case2.dev.workspace)
    torch.cuda.synchronize()
    assert syncs == B.spd_sync_count(case2.dev.ctx, w.mask) == 5
    assert np.max(np.abs(out2.cpu().numpy() - chain)) <= 2e-3
    chain = out2.cpu().numpy()
    want = O.model_single_rank(case2.sh, X, [s[0] for s in case2.shards], [c[0] for c in case2.caches], positions,
                               batch, q_len, w.mask, rank, peers.astype(np.float64))
    err = float(np.max(np.abs(chain - want)))
    rms = float(np.sqrt(np.mean(want ** 2)))
    say(f"mid end-to-end over {w.n_layers} layers: max err {err:.2e}, output rms {rms:.2f}")
    assert err <= 2e-2 * w.n_layers * max(1.0, rms)
    # run twice: bit-identical (fixed summation orders, no float atomics)
    case3 = Case(w, gpu, ranks=[rank], positions=positions, max_ctx=256, max_tokens=48)
    out3 = torch.empty_like(out2)
    B.spd_model_forward(case3.dev.ctx, w.mask, rank, case3.dev.weights, case3.dev.kv, positions, batch, q_len,
                        case3.to_dev(X), case3.to_dev(peers), out3, case3.dev.workspace)
    torch.cuda.synchronize()
    assert np.array_equal(out3.cpu().numpy(), chain)
    for c in (case, case2, case3):
        c.close()


def test_bf16_prefill_then_decode_matches_longer_prefill(gpu):
    """KV-cache consistency on the device: 20 tokens at once == 12 at once + 8 one by one."""
    import torch
    w = SMALL
    X = inputs.hidden_states(w, 20)
    full = Case(w, gpu, ranks=range(w.tp), positions=[0], max_ctx=64, max_tokens=32)
    slots = torch.zeros((w.tp, 20, w.hidden), dtype=torch.float32, device=gpu)
    o_full = torch.empty((20, w.hidden), dtype=torch.float32, device=gpu)
    B.spd_model_forward(full.dev.ctx, w.mask, B.SPD_ALL_RANKS, full.dev.weights, full.dev.kv, [0], 1, 20,
                        full.to_dev(X), slots, o_full, full.dev.workspace)
    step = Case(w, gpu, ranks=range(w.tp), positions=[0], max_ctx=64, max_tokens=32)
    o_head = torch.empty((12, w.hidden), dtype=torch.float32, device=gpu)
    B.spd_model_forward(step.dev.ctx, w.mask, B.SPD_ALL_RANKS, step.dev.weights, step.dev.kv, [0], 1, 12,
                        step.to_dev(X[:12]), slots, o_head, step.dev.workspace)
    torch.cuda.synchronize()
    want, _ = O.model_all_ranks(full.sh, X, full.shards, full.caches, [0], 1, 20, w.mask)
    assert_close(o_full.cpu().numpy(), want, w, "20-token chunk")
    assert_close(o_head.cpu().numpy(), want[:12], w, "12-token chunk")
    for t in range(12, 20):
        o1 = torch.empty((1, w.hidden), dtype=torch.float32, device=gpu)
        B.spd_model_forward(step.dev.ctx, w.mask, B.SPD_ALL_RANKS, step.dev.weights, step.dev.kv, [t], 1, 1,
                            step.to_dev(X[t:t + 1]), slots, o1, step.dev.workspace)
        torch.cuda.synchronize()
        assert_close(o1.cpu().numpy()[0], want[t], w, f"step {t}")
    full.close()
    step.close()


def test_edge_cases(gpu):
    import torch
    w = SMALL
    # maximum position: the last slot of the cache; and maximum batch
    case = Case(w, gpu, ranks=[1], positions=[63, 0, 63], max_ctx=64, max_tokens=16)
    X = inputs.hidden_states(w, 3)
    peers = inputs.peer_slots(w, 3)
    slots = case.to_dev(peers)
    out = torch.empty((3, w.hidden), dtype=torch.float32, device=gpu)
    B.spd_block_forward(case.dev.ctx, 0, 1, 1, case.dev.weights[0], case.dev.kv[0], [63, 0, 63], 3, 1,
                        case.to_dev(X), slots, out, case.dev.workspace)
    torch.cuda.synchronize()
    want = O.block_single_rank(case.sh, X, case.shards[0][0], case.caches[0][0], [63, 0, 63], 3, 1, 1, 1,
                               peers.astype(np.float64))
    assert_close(out.cpu().numpy(), want, w, "max position")
    # empty call: nothing is launched, the output buffer is left alone
    out.fill_(5.0)
    B.spd_block_forward(case.dev.ctx, 0, 1, 1, case.dev.weights[0], case.dev.kv[0], [], 0, 1,
                        case.to_dev(X), slots, out, case.dev.workspace)
    torch.cuda.synchronize()
    assert float(out.min()) == 5.0
    # x_out may alias x_in
    x = case.to_dev(X)
    case_b = Case(w, gpu, ranks=[1], positions=[63, 0, 63], max_ctx=64, max_tokens=16)
    B.spd_block_forward(case_b.dev.ctx, 0, 0, 1, case_b.dev.weights[0], case_b.dev.kv[0], [63, 0, 63], 3, 1,
                        x, case_b.to_dev(peers), x, case_b.dev.workspace)
    torch.cuda.synchronize()
    want = O.block_single_rank(case_b.sh, X, case_b.shards[0][0], case_b.caches[0][0], [63, 0, 63], 3, 1, 0, 1,
                               peers.astype(np.float64))
    assert_close(x.cpu().numpy(), want, w, "aliased output")
    case.close()
    case_b.close()
    # 64 sequences in one call
    w64 = Workload(name="b64", hidden=128, n_q_heads=4, n_kv_heads=2, head_dim=32, ffn=128, n_layers=1, tp=2,
                   dtype=BF16, seed=14, batch=64, q_len=1, ctx=32, mask=(1,))
    pos = [(7 * i) % 32 for i in range(64)]
    c64 = Case(w64, gpu, ranks=range(2), positions=pos, max_ctx=32, max_tokens=64)
    X = inputs.hidden_states(w64, 64)
    slots = torch.zeros((2, 64, 128), dtype=torch.float32, device=gpu)
    out = torch.empty((64, 128), dtype=torch.float32, device=gpu)
    B.spd_block_forward(c64.dev.ctx, 0, 1, B.SPD_ALL_RANKS, c64.dev.weights[0], c64.dev.kv[0], pos, 64, 1,
                        c64.to_dev(X), slots, out, c64.dev.workspace)
    torch.cuda.synchronize()
    want, _ = O.block_all_ranks(c64.sh, X, c64.shards[0], c64.caches[0], pos, 64, 1, 1)
    assert_close(out.cpu().numpy(), want, w64, "64 sequences")
    c64.close()


def test_long_context_decode(gpu):
    """Decode steps against caches of 16383, 9000 and 31 positions in one call (capacity 16384): the attention
    kernel cuts the context into as many splits as it may and merges them; one rank of four."""
    import torch
    w, rank = SMALL, 2
    positions = [16383, 9000, 31]
    case = Case(w, gpu, ranks=[rank], positions=positions, max_ctx=16384, max_tokens=16)
    X = inputs.hidden_states(w, 3)
    peers = inputs.peer_slots(w, 3)
    slots = case.to_dev(peers)
    out = torch.empty((3, w.hidden), dtype=torch.float32, device=gpu)
    say("long-context decode, positions", positions)
    for l, flag in enumerate(w.mask):
        x_in = X if l == 0 else out.cpu().numpy()
        B.spd_block_forward(case.dev.ctx, l, flag, rank, case.dev.weights[l], case.dev.kv[l], positions, 3, 1,
                            case.to_dev(x_in), slots, out, case.dev.workspace)
        torch.cuda.synchronize()
        want = O.block_single_rank(case.sh, x_in, case.shards[l][0], case.caches[l][0], positions, 3, 1, flag, rank,
                                   peers.astype(np.float64))
        err = assert_close(out.cpu().numpy(), want, w, f"long context block {l}")
        say(f"  block {l}: max err {err:.2e}")
    case.close()


# ------------------------------------------------------------------------------------------------
# full-size shapes through spd_block_forward (2 layers each: the first as an SPD block, the last as a TP block);
# the call the bench makes, spd_model_forward at full depth, is checked at the end of this file
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("name", ["7b-decode", "13b-decode", "70b-decode", "7b-tp4-decode", "13b-tp4-decode"])
def test_full_size_decode_shapes(gpu, name):
    import torch
    full = workloads.get(name)
    w = full.with_layers(2).with_mask((1, 0))
    layer_ids = [0, full.n_layers - 1]
    positions = [full.ctx - 1] * full.batch
    say(f"full-size {name}: batch {full.batch}, ctx {full.ctx}")
    case = Case(w, gpu, ranks=[0], positions=positions, layer_ids=layer_ids)
    M = full.batch
    X = inputs.hidden_states(w, M)
    peers = inputs.peer_slots(w, M)
    x = case.to_dev(X)
    slots = case.to_dev(peers)
    for l in range(2):
        x_host = x.cpu().numpy()
        out = torch.empty_like(x)
        B.spd_block_forward(case.dev.ctx, l, w.mask[l], 0, case.dev.weights[l], case.dev.kv[l], positions, M, 1, x,
                            slots, out, case.dev.workspace)
        torch.cuda.synchronize()
        want = O.block_single_rank(case.sh, x_host, case.shards[l][0], case.caches[l][0], positions, M, 1, w.mask[l],
                                   0, peers.astype(np.float64))
        err = assert_close(out.cpu().numpy(), want, w, f"{name} layer {layer_ids[l]} flag {w.mask[l]}")
        say(f"  layer {layer_ids[l]} flag {w.mask[l]}: max err {err:.2e}, max |oracle| {np.max(np.abs(want)):.2f}")
        x = out
    case.close()


@pytest.mark.parametrize("batch", [24, 48, 64])
def test_full_size_large_batch_decode(gpu, batch):
    """LLaMA2-70B shard, one decode step of 24 / 48 / 64 sequences at ragged positions of a 1024-position cache: the
    projections take the kernels for 17 to 512 tokens, the QKV one on a single activation plane (a decode step
    attends to one new key per sequence).  An SPD block and a TP block, every row at the 2e-2 bound."""
    import torch
    from dataclasses import replace
    full = replace(workloads.get("70b-decode"), batch=batch, ctx=1024)
    w = full.with_layers(2).with_mask((1, 0))
    positions = [int(p) for p in np.random.default_rng(batch).integers(0, full.ctx, size=batch)]
    positions[0], positions[-1] = full.ctx - 1, 0
    say(f"full-size decode, batch {batch}")
    case = Case(w, gpu, ranks=[0], positions=positions, layer_ids=[0, workloads.get("70b-decode").n_layers - 1])
    X = inputs.hidden_states(w, batch)
    peers = inputs.peer_slots(w, batch)
    x, slots = case.to_dev(X), case.to_dev(peers)
    for l in range(2):
        x_host = x.cpu().numpy()
        out = torch.empty_like(x)
        B.spd_block_forward(case.dev.ctx, l, w.mask[l], 0, case.dev.weights[l], case.dev.kv[l], positions, batch, 1, x,
                            slots, out, case.dev.workspace)
        torch.cuda.synchronize()
        want = O.block_single_rank(case.sh, x_host, case.shards[l][0], case.caches[l][0], positions, batch, 1, w.mask[l],
                                   0, peers.astype(np.float64))
        err = assert_close(out.cpu().numpy(), want, w, f"decode batch {batch} flag {w.mask[l]}")
        say(f"  flag {w.mask[l]}: max err {err:.2e}, max |oracle| {np.max(np.abs(want)):.2f}")
        x = out
    case.close()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("q_len", [128, 200, 500])
def test_full_size_short_prefill(gpu, q_len):
    """LLaMA2-70B shard, one sequence of 128 tokens (the shape of the paper's latency breakdown,
    Fig. 2), an SPD block then a TP block, every output row checked at the 2e-2 bound as it
    stands, in the default configuration (the one the bench times).  200 and 500 tokens: from 145
    tokens on the QKV and down projections take the kernel that shares the activations through LDS
    (the QKV one on its hi + lo input pair), with ragged last m-tiles."""
    import torch
    from dataclasses import replace
    full = workloads.get("70b-prefill-128")
    full = replace(full, q_len=q_len, ctx=(q_len + 31) // 32 * 32)
    w = full.with_layers(2).with_mask((1, 0))
    M = full.q_len
    case = Case(w, gpu, ranks=[0], positions=[0], layer_ids=[0, full.n_layers - 1])
    X = inputs.hidden_states(w, M)
    peers = inputs.peer_slots(w, M)
    x, slots = case.to_dev(X), case.to_dev(peers)
    say(f"full-size short prefill: 1 x {M} tokens")
    for l in range(2):
        x_host = x.cpu().numpy()
        out = torch.empty_like(x)
        B.spd_block_forward(case.dev.ctx, l, w.mask[l], 0, case.dev.weights[l], case.dev.kv[l], [0], 1, M, x, slots, out,
                            case.dev.workspace)
        torch.cuda.synchronize()
        want = O.block_single_rank(case.sh, x_host, case.shards[l][0], case.caches[l][0], [0], 1, M, w.mask[l], 0,
                                   peers.astype(np.float64))
        err = assert_close(out.cpu().numpy(), want, w, f"short prefill layer {l}")
        say(f"  flag {w.mask[l]}: max err {err:.2e}, max |oracle| {np.max(np.abs(want)):.2f}")
        x = out
    # the same two blocks through spd_model_forward (the call the bench makes: the down projection's epilogue then
    # carries the closing sync point and the next block's norm preparation), block by block against the oracle
    case2 = Case(w, gpu, ranks=[0], positions=[0], layer_ids=[0, full.n_layers - 1])
    taps = torch.zeros((2, M, w.hidden), dtype=torch.float32, device=gpu)
    out2 = torch.empty((M, w.hidden), dtype=torch.float32, device=gpu)
    syncs = B.spd_model_forward_staged(case2.dev.ctx, w.mask, 0, case2.dev.weights, case2.dev.kv, [0], 1, M, case2.to_dev(X),
                                       case2.to_dev(peers), out2, case2.dev.workspace, layer_out=taps)
    torch.cuda.synchronize()
    assert syncs == 3
    got = taps.cpu().numpy()
    for l in range(2):
        x_in = X if l == 0 else got[l - 1]
        want = O.block_single_rank(case2.sh, x_in, case2.shards[l][0], case2.caches[l][0], [0], 1, M, w.mask[l], 0,
                                   peers.astype(np.float64))
        err = assert_close(got[l], want, w, f"short prefill, model forward, layer {l}")
        say(f"  model forward, flag {w.mask[l]}: max err {err:.2e}")
    case2.close()
    case.close()


@pytest.mark.parametrize("q_len", [700, 1100, 2048])
def test_full_size_single_sequence_prefill(gpu, q_len):
    """LLaMA2-70B shard, one sequence of 700 / 1100 / 2048 tokens: a single chain, whose QKV GEMM has too few tiles
    for 256 compute units and runs in K slices side by side, whose partial rows a finishing kernel adds;
    at 700 tokens the other projections run as 256 x 128 half tiles throughout (a ragged last one).  An SPD
    block and a TP block, sampled output rows against the oracle at 2e-2."""
    import torch
    from dataclasses import replace
    full = replace(workloads.LLAMA70B_PREFILL, batch=1, q_len=q_len, ctx=(q_len + 31) // 32 * 32)
    w = full.with_layers(2).with_mask((1, 0))
    M = q_len
    rows = np.unique(np.concatenate([np.array([0, 1, 15, 16, 255, 256, 511, 512, 640, M - 17, M - 1]),
                                     np.random.default_rng(5).choice(M, size=54, replace=False)]))
    X = inputs.hidden_states(w, M)
    peers = inputs.peer_slots(w, M)
    say(f"full-size single-sequence prefill: 1 x {M} tokens")
    case = Case(w, gpu, ranks=[0], positions=[0], layer_ids=[0, workloads.LLAMA70B_PREFILL.n_layers - 1])
    x, slots = case.to_dev(X), case.to_dev(peers)
    sel = torch.from_numpy(rows).to(gpu)
    for l in range(2):
        x_host = x.cpu().numpy()
        out = torch.empty_like(x)
        B.spd_block_forward(case.dev.ctx, l, w.mask[l], 0, case.dev.weights[l], case.dev.kv[l], [0], 1, M, x, slots, out,
                            case.dev.workspace)
        torch.cuda.synchronize()
        want = O.block_single_rank(case.sh, x_host, case.shards[l][0], case.caches[l][0], [0], 1, M, w.mask[l], 0,
                                   peers.astype(np.float64), rows=rows)
        err = assert_close(out[sel].cpu().numpy(), want, w, f"single-sequence prefill layer {l}")
        say(f"  flag {w.mask[l]}: max err {err:.2e} on {len(rows)} sampled rows")
        assert bool(torch.isfinite(out).all())
        x = out
    # the appended keys and values of the first block, all positions: bf16 copies of the oracle's
    k, v = case.dev.read_kv(0, 0, 1, M)
    ko, vo = case.caches[0][0].k[0, :, :M], case.caches[0][0].v[0, :, :M]
    assert np.max(np.abs(k[0] - ko)) <= 2.0 ** -7 * np.max(np.abs(ko)) + 1e-3
    assert np.max(np.abs(v[0] - vo)) <= 2.0 ** -7 * np.max(np.abs(vo)) + 1e-3
    case.close()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("flag", [1, 0], ids=["spd", "tp"])
@pytest.mark.parametrize("split", [B.SPD_SPLIT_AUTO, B.SPD_SPLIT_ALWAYS], ids=["default", "all-split"])
def test_full_size_prefill_shape_sampled_rows(gpu, flag, split):
    """LLaMA2-70B shard, 4 x 2048 tokens, the launch configuration the bench times (and, beside
    it, the one with every projection input split): the oracle computes sampled output rows one
    by one; the 2e-2 bound as it stands."""
    import torch
    full = workloads.LLAMA70B_PREFILL
    w = full.with_layers(1).with_mask((flag,))
    M = full.batch * full.q_len
    rows = np.unique(np.concatenate([
        np.array([0, 1, 15, 16, 17, 255, 256, 2047, 2048, 2049, 3000, 4095, 4096, 5555, 6143, 6144, 8000, 8191]),
        np.random.default_rng(7).choice(M, size=110, replace=False)]))
    X = inputs.hidden_states(w, M)
    peers = inputs.peer_slots(w, M)
    say(f"full-size prefill flag={flag} split={split}")
    case = Case(w, gpu, ranks=[0], positions=[0] * full.batch, act_split=split)
    x = case.to_dev(X)
    slots = case.to_dev(peers)
    out = torch.empty_like(x)
    B.spd_block_forward(case.dev.ctx, 0, flag, 0, case.dev.weights[0], case.dev.kv[0], [0] * full.batch,
                        full.batch, full.q_len, x, slots, out, case.dev.workspace)
    torch.cuda.synchronize()
    got = out[torch.from_numpy(rows).to(gpu)].cpu().numpy()
    del x, out
    want = O.block_single_rank(case.sh, X, case.shards[0][0], case.caches[0][0], [0] * full.batch, full.batch,
                               full.q_len, flag, 0, peers, rows=rows)
    rms = float(np.sqrt(np.mean(want ** 2)))
    worst = np.max(np.abs(got - want), axis=1)
    say("  largest per-row max err:", " ".join(f"{rows[i]}:{worst[i]:.1e}" for i in np.argsort(worst)[-6:]))
    err = assert_close(got, want, w, f"prefill rows flag={flag} split={split}")
    say(f"  {len(rows)} sampled rows: max err {err:.2e}, max |oracle| {np.max(np.abs(want)):.2f}, rms {rms:.2f}")
    if split == B.SPD_SPLIT_AUTO:
        # what the bench launches: spd_model_forward (two chains of 2 x 2048 tokens on two streams) replayed from a
        # HIP graph; the same sampled rows against the same oracle rows
        x = case.to_dev(X)
        slots_g = case.to_dev(peers)
        out_g = torch.empty_like(x)
        graph = _capture(torch, lambda: B.spd_model_forward(case.dev.ctx, w.mask, 0, case.dev.weights, case.dev.kv,
                                                            [0] * full.batch, full.batch, full.q_len, x, slots_g, out_g,
                                                            case.dev.workspace))
        out_g.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        got_g = out_g[torch.from_numpy(rows).to(gpu)].cpu().numpy()
        err_g = assert_close(got_g, want, w, f"prefill rows, two chains under a graph, flag={flag}")
        say(f"  two chains replayed from a graph: max err {err_g:.2e}; against the one-chain block call {np.max(np.abs(got_g - got)):.2e}")
        assert bool(torch.isfinite(out_g).all())
        del graph, x, out_g, slots_g
    # properties that hold at any size: peers' slots untouched; finite everywhere
    assert np.array_equal(slots[5][:64].cpu().numpy(), peers[5][:64])
    assert bool(torch.isfinite(slots[0]).all())
    del slots
    case.close()
    torch.cuda.empty_cache()


# ------------------------------------------------------------------------------------------------
# the prefill call the bench makes, several blocks deep: two chains, each block's closing sync point
# preparing the next block's first norm
# ------------------------------------------------------------------------------------------------
def test_full_size_prefill_model_forward_three_blocks(gpu):
    """LLaMA2-70B shard, 4 x 2048 tokens through spd_model_forward (two chains of 2 x 2048 on two streams) over
    three blocks with mask (1, 0, 1): every block's output on sampled rows against the oracle's block fed the
    input the library's block had (all rows of it: the keys and values of every token matter), 2e-2 each."""
    import torch
    full = workloads.LLAMA70B_PREFILL
    w = full.with_layers(3).with_mask((1, 0, 1))
    batch, q_len = full.batch, full.q_len
    M = batch * q_len
    positions = [0] * batch
    rows = np.unique(np.concatenate([np.array([0, 15, 16, 2047, 2048, 4095, 4096, 6144, 8191]),
                                     np.random.default_rng(11).choice(M, size=40, replace=False)]))
    X = inputs.hidden_states(w, M)
    peers = inputs.peer_slots(w, M)
    say(f"full-size prefill, model forward over {w.n_layers} blocks, mask {w.mask}")
    case = Case(w, gpu, ranks=[0], positions=positions)
    x, slots = case.to_dev(X), case.to_dev(peers)
    out = torch.empty_like(x)
    taps = torch.zeros((w.n_layers, M, w.hidden), dtype=torch.float32, device=gpu)
    syncs = B.spd_model_forward_staged(case.dev.ctx, w.mask, 0, case.dev.weights, case.dev.kv, positions, batch, q_len, x,
                                       slots, out, case.dev.workspace, layer_out=taps)
    torch.cuda.synchronize()
    assert syncs == B.spd_sync_count(case.dev.ctx, w.mask) == 4
    assert bool(torch.equal(taps[-1], out))
    sel = torch.from_numpy(rows).to(gpu)
    worst = 0.0
    for l in range(w.n_layers):
        x_in = X if l == 0 else taps[l - 1].cpu().numpy()
        want = O.block_single_rank(case.sh, x_in, case.shards[l][0], case.caches[l][0], positions, batch, q_len,
                                   int(w.mask[l]), 0, peers.astype(np.float64), rows=rows)
        err = assert_close(taps[l][sel].cpu().numpy(), want, w, f"prefill model forward block {l} (mask {w.mask[l]})")
        say(f"  block {l}: max err {err:.2e} on {len(rows)} sampled rows")
        worst = max(worst, err)
    del taps, x, out, slots
    case.close()
    torch.cuda.empty_cache()


# ------------------------------------------------------------------------------------------------
# the call the bench makes: spd_model_forward at full depth with the workload's own mask
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("name,n_syncs", [("7b-decode", 32), ("13b-decode", 50), ("70b-decode", 96)])
def test_full_depth_model_forward(gpu, name, n_syncs):
    """Rank 0's share of the whole model (32 / 40 / 80 blocks, the workload's mask: all SPD, every 4th
    block synced, SPD on blocks 8..71) through spd_model_forward, the call the bench times, where each
    block's closing sync point also prepares the next block's first norm.  Every block's output is
    compared with the oracle's block fed the same input (2e-2 as it stands); the whole chain is compared
    with the oracle's own chain relative to the output's rms."""
    import torch
    w = workloads.get(name)
    M, positions = w.batch, [w.ctx - 1] * w.batch
    say(f"full depth {name}: {w.n_layers} blocks, mask sum {sum(w.mask)}, batch {w.batch}, ctx {w.ctx}")
    dev = B.DeviceShard(w, [0], gpu)
    n_pre = w.ctx - 1
    for l in range(w.n_layers):
        dev.load_layer(l, [inputs.layer_shard(w, l, 0)])
        dev.load_kv(l, [inputs.kv_prefill(w, l, 0, w.batch, n_pre)])
    X = inputs.hidden_states(w, M)
    peers = inputs.peer_slots(w, M)
    x, slots = torch.from_numpy(X).to(gpu), torch.from_numpy(peers).to(gpu)
    out = torch.empty_like(x)
    taps = torch.zeros((w.n_layers, M, w.hidden), dtype=torch.float32, device=gpu)
    syncs = B.spd_model_forward_staged(dev.ctx, w.mask, 0, dev.weights, dev.kv, positions, w.batch, 1, x, slots, out,
                                       dev.workspace, layer_out=taps)
    torch.cuda.synchronize()
    assert syncs == B.spd_sync_count(dev.ctx, w.mask) == n_syncs
    got = taps.cpu().numpy()
    assert np.array_equal(got[-1], out.cpu().numpy())
    # the launch configuration the bench times: the same call replayed from a HIP graph (twice, into another
    # output buffer) gives the eager result bit for bit
    out_g = torch.empty_like(x)
    slots_g = torch.from_numpy(peers).to(gpu)
    graph = _capture(torch, lambda: B.spd_model_forward(dev.ctx, w.mask, 0, dev.weights, dev.kv, positions, w.batch, 1, x,
                                                        slots_g, out_g, dev.workspace))
    for rep in range(2):
        out_g.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out_g.cpu().numpy(), got[-1]), f"graph replay {rep} differs from the eager forward"
    del graph
    dev.close()
    del dev, taps
    torch.cuda.empty_cache()

    sh = oracle_shapes(w)
    mc = (w.ctx + 31) // 32 * 32
    o_slots = peers.astype(np.float64)
    chain = X.astype(np.float64)
    worst, worst_l = 0.0, -1
    for l in range(w.n_layers):
        shard = inputs.layer_shard(w, l, 0)
        k, v = inputs.kv_prefill(w, l, 0, w.batch, n_pre)
        cache = O.KVCache(w.batch, w.kv_per_rank, mc, w.head_dim, storage=cache_storage(w))
        cache.fill(k, v)
        x_in = X if l == 0 else got[l - 1]
        want = O.block_single_rank(sh, x_in, shard, cache.copy(), positions, w.batch, 1, int(w.mask[l]), 0, o_slots)
        err = assert_close(got[l], want, w, f"{name} block {l} (mask {w.mask[l]})")
        if err > worst:
            worst, worst_l = err, l
        chain = O.block_single_rank(sh, chain, shard, cache, positions, w.batch, 1, int(w.mask[l]), 0, o_slots)
    rms = float(np.sqrt(np.mean(chain ** 2)))
    e2e = float(np.max(np.abs(got[-1] - chain)))
    say(f"  worst block {worst_l}: max err {worst:.2e}; end to end: max err {e2e:.2e}, output rms {rms:.2f}, "
        f"relative {e2e / rms:.2e}")
    # errors of the blocks add up along the chain (each at most 2e-2, amplified or damped by what follows):
    # the end-to-end figure is reported relative to the output's rms and bounded by the sum of the per-block bounds
    assert e2e <= 2e-2 * w.n_layers * max(1.0, rms)


# ------------------------------------------------------------------------------------------------
# a long prefill of several sequences: spd_model_forward runs it as two chains on two streams
# ------------------------------------------------------------------------------------------------
TWO_CHAIN = Workload(name="two-chain-bf16", hidden=256, n_q_heads=8, n_kv_heads=4, head_dim=64, ffn=832, n_layers=3,
                     tp=4, dtype=BF16, seed=19, batch=3, q_len=1100, ctx=1120, mask=(1, 0, 1))


def test_bf16_two_chain_prefill(gpu):
    """Three sequences of 1100 tokens (the second one continuing after 5 cached positions): the model
    forward cuts the call into a chain of two sequences and a chain of one and runs them on two streams.
    Every block's output is checked against the oracle's block fed the same input, and the result against
    what the blocks give one after the other on one stream (spd_block_forward)."""
    import torch
    w, rank = TWO_CHAIN, 1
    batch, q_len, positions = w.batch, w.q_len, [0, 5, 0]
    M = batch * q_len
    X = inputs.hidden_states(w, M)
    peers = inputs.peer_slots(w, M)
    case = Case(w, gpu, ranks=[rank], positions=positions, max_ctx=w.ctx, max_tokens=M)
    x, slots = case.to_dev(X), case.to_dev(peers)
    out = torch.empty_like(x)
    taps = torch.zeros((w.n_layers, M, w.hidden), dtype=torch.float32, device=gpu)
    say(f"two-chain prefill: {batch} x {q_len} tokens")
    syncs = B.spd_model_forward_staged(case.dev.ctx, w.mask, rank, case.dev.weights, case.dev.kv, positions, batch, q_len,
                                       x, slots, out, case.dev.workspace, layer_out=taps)
    torch.cuda.synchronize()
    assert syncs == B.spd_sync_count(case.dev.ctx, w.mask) == 4
    got = taps.cpu().numpy()
    assert np.array_equal(got[-1], out.cpu().numpy())
    # the same blocks one after the other, one chain
    ref = Case(w, gpu, ranks=[rank], positions=positions, max_ctx=w.ctx, max_tokens=M)
    xr, sr = ref.to_dev(X), ref.to_dev(peers)
    for l in range(w.n_layers):
        o = torch.empty_like(xr)
        B.spd_block_forward(ref.dev.ctx, l, w.mask[l], rank, ref.dev.weights[l], ref.dev.kv[l], positions, batch, q_len, xr,
                            sr, o, ref.dev.workspace)
        xr = o
    torch.cuda.synchronize()
    # (not bit for bit: which kernel runs a projection depends on the number of tokens of the call or chain, and
    # the kernels add up K in different orders)
    d = float(np.max(np.abs(xr.cpu().numpy() - got[-1])))
    say(f"  two chains vs one chain of blocks: max difference {d:.2e}")
    assert d <= 2e-3
    assert float(np.max(np.abs(sr.cpu().numpy() - slots.cpu().numpy()))) <= 2e-3
    for l in (0, w.n_layers - 1):
        k0, v0 = case.dev.read_kv(l, 0, batch, max(positions) + q_len)
        k1, v1 = ref.dev.read_kv(l, 0, batch, max(positions) + q_len)
        # bf16 values on both sides; a last-bit disagreement is one unit in the last place
        assert np.max(np.abs(k0 - k1)) <= 2.0 ** -7 * np.max(np.abs(k1)) and np.max(np.abs(v0 - v1)) <= 2.0 ** -7 * np.max(np.abs(v1))
    ref.close()
    # block by block against the oracle
    o_slots = peers.astype(np.float64)
    worst = 0.0
    for l in range(w.n_layers):
        x_in = X if l == 0 else got[l - 1]
        want = O.block_single_rank(case.sh, x_in, case.shards[l][0], case.caches[l][0], positions, batch, q_len, w.mask[l],
                                   rank, o_slots)
        worst = max(worst, assert_close(got[l], want, w, f"two-chain block {l}"))
    say(f"  worst block max err {worst:.2e}")
    case.close()


# ------------------------------------------------------------------------------------------------
# bench.py names the kernels of the gate/up stage it times (and takes their traffic and durations from profiles/ by that name): the names against
# those of the launches, as a profiler sees them, on every model's shard from one token to two chains
def _kernel_label(name):
    """k_name<arguments> of a kernel's mangled or demangled name."""
    import re
    m = re.match(r"_ZN12_GLOBAL__N_1(\d+)", name)
    if not m:
        return re.sub(r"\(anonymous namespace\)::|^void | ", "", name).split("(")[0]
    n = int(m[1])
    base, rest, args = name[m.end():m.end() + n], name[m.end() + n + 1:], []
    while (t := re.match(r"Li(\d+)E|Lb([01])E|NS_(\d+)", rest)):
        rest = rest[t.end():]
        if t[3]:
            args.append(rest[:int(t[3])])
            rest = rest[int(t[3]) + 1:]
        else:
            args.append(t[1] or ("true" if t[2] == "1" else "false"))
    return f"{base}<{','.join(args)}>"


@pytest.mark.parametrize("model", ["7b-decode", "13b-decode", "70b-decode", "7b-tp4-decode", "13b-tp4-decode"])
def test_bench_names_the_kernels_it_times(gpu, model):
    import torch
    from dataclasses import replace
    from torch.profiler import ProfilerActivity, profile

    import bench
    base = workloads.get(model)
    shapes = [(1, 1), (16, 1), (17, 1), (64, 1)] + [(1, n) for n in (24, 48, 100, 128, 129, 200, 333, 512, 513, 600, 760, 1000, 1500, 2048, 3000, 4096)]
    shapes += [(2, 1024), (4, 2048)]
    most = max(b * q for b, q in shapes)
    shard = B.DeviceShard(replace(base, n_layers=1, mask=(1,)), [0], gpu, max_ctx=4096, max_tokens=most, max_batch=64)
    shard.weights[0].zero_()
    x = torch.zeros((most, base.hidden), dtype=torch.float32, device=gpu)
    slots, out = torch.zeros((base.tp, most, base.hidden), dtype=torch.float32, device=gpu), torch.empty_like(x)

    def call(b, q):
        B.spd_model_forward_staged(shard.ctx, (1,), 0, shard.weights, shard.kv, [0] * b, b, q, x[:b * q], slots.view(-1)[:base.tp * b * q * base.hidden],
                                   out[:b * q], shard.workspace, stage_mask=1 << B.STAGES["gateup"])

    call(1, 1)
    torch.cuda.synchronize()
    for b, q in shapes:
        with profile(activities=[ProfilerActivity.CUDA, ProfilerActivity.CPU]) as prof:
            for _ in range(3):           # (the profiler loses a launch now and then)
                call(b, q)
            torch.cuda.synchronize()
        names = [_kernel_label(e.name) for e in prof.events() if e.device_type != torch.autograd.DeviceType.CPU]
        names = {n for n in names if n.startswith(("k_gemv", "k_mid", "k_skinny", "k_gemm_lds"))}
        label = bench.stage_kernel(replace(base, batch=b, q_len=q), "gateup")
        say(f"{model} {b} x {q}: {label}")
        assert names == set(label.replace("x2", "").split("+")), (model, b, q, names, label)
    shard.close()


# the launch configuration bench.py times: the whole-model forward replayed from a HIP graph
# ------------------------------------------------------------------------------------------------
def _capture(torch, fn):
    """fn() captured into a graph on a side stream, the way bench.py does it."""
    stream = torch.cuda.current_stream()
    side = torch.cuda.Stream()
    side.wait_stream(stream)
    with torch.cuda.stream(side):
        fn()
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            fn()
    stream.wait_stream(side)
    torch.cuda.synchronize()
    return graph


@pytest.mark.parametrize("kind", ["decode", "two-chain-prefill"])
def test_graph_replays_equal_the_eager_forward(gpu, kind):
    """spd_model_forward captured into a HIP graph and replayed three times, each time on new hidden states written
    into the same buffers, with the library's own eager forward between the replays: every replay must equal the
    eager result on the same inputs bit for bit (the path is deterministic).  The two-chain prefill records
    its second chain on the library's helper stream into the same graph."""
    import torch
    if kind == "decode":
        w, rank, batch, q_len = MID, 3, 2, 1
        positions = [100, 37]
        case = Case(w, gpu, ranks=[rank], positions=positions, max_ctx=256, max_tokens=48)
    else:
        w, rank, batch, q_len = TWO_CHAIN, 1, TWO_CHAIN.batch, TWO_CHAIN.q_len
        positions = [0, 5, 0]
        case = Case(w, gpu, ranks=[rank], positions=positions, max_ctx=w.ctx, max_tokens=batch * q_len)
    M = batch * q_len
    X = inputs.hidden_states(w, M)
    peers = inputs.peer_slots(w, M)
    x = case.to_dev(X)
    slots, slots_e = case.to_dev(peers), case.to_dev(peers)
    out, out_e = torch.empty_like(x), torch.empty_like(x)

    def run(o, sl):
        return B.spd_model_forward(case.dev.ctx, w.mask, rank, case.dev.weights, case.dev.kv, positions, batch, q_len, x, sl, o,
                                   case.dev.workspace)

    graph = _capture(torch, lambda: run(out, slots))
    for rep in range(3):
        say(f"graph replay {rep} ({kind})")
        x.copy_(torch.from_numpy(X * (1.0 + 0.25 * rep)).to(gpu))         # new inputs in the captured buffers
        out.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        got, got_slot = out.cpu().numpy().copy(), slots[rank].cpu().numpy().copy()
        out_e.fill_(-2.0)
        run(out_e, slots_e)                                                # eager, same inputs, other output buffers
        torch.cuda.synchronize()
        assert np.isfinite(got).all()
        assert np.array_equal(got, out_e.cpu().numpy()), f"replay {rep} differs from the eager forward"
        assert np.array_equal(got_slot, slots_e[rank].cpu().numpy())
    case.close()


@pytest.mark.gpu
def test_mfma_probe_reports_a_plausible_rate():
    """The benchmark aid runs and lands between a tenth of and the whole nominal fp16 MFMA peak, at a clock the chip has."""
    import torch
    scratch = torch.empty(B.SPD_MFMA_PROBE_SCRATCH_BYTES, dtype=torch.uint8, device="cuda:0")
    for random_data in (True, False):
        tf, mhz = B.spd_mfma_probe(2000, random_data, scratch)
        assert 250.0 < tf < 2600.0, (random_data, tf)
        assert 500.0 < mhz < 2600.0, (random_data, mhz)


def test_read_probe_reports_a_plausible_rate(gpu):
    """The benchmark aid runs: 64 MiB per launch from 8 distinct buffers, between 1 and 8 TB/s."""
    import torch
    chunk = 64 << 20
    buf = torch.zeros(8 * chunk, dtype=torch.uint8, device=gpu)
    sink = torch.zeros(4, dtype=torch.float32, device=gpu)
    us = B.spd_read_probe(buf, chunk, 8, 16, sink)
    rate = chunk / (us * 1e-6) / 1e12
    say(f"read probe: {us:.2f} us per 64 MiB = {rate:.2f} TB/s")
    assert 1.0 < rate < 8.0
    assert float(sink.sum()) == 0.0
