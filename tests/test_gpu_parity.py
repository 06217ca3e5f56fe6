"""GPU parity: every C-ABI entry point against the CPU fp64 oracle, element by
element, on seeded inputs that span several tiles and a ragged tail."""
import itertools

import numpy as np
import pytest
import torch

import paper_2407_21018_amd as thk
from oracle import oracle as O
from paper_2407_21018_amd.synth import as_numpy
from helpers import (ATTN_TOL, DT, SCORE_TOL, TDT, attn_rel_err, check_idx_with_tie_rule, gpu_compact,
                     gpu_decode, gpu_prune, gpu_score, gpu_select, oracle_prune, ws_tensor)

pytestmark = pytest.mark.gpu
D = 128


def _randn(shape, dtype, seed, scale_sigma=1.0, dev="cuda"):
    g = torch.Generator(device=dev); g.manual_seed(seed)
    x = torch.randn(*shape, generator=g, device=dev)
    if scale_sigma:
        sc = torch.exp(scale_sigma * torch.randn(shape[-1], generator=g, device=dev))
        x = x * sc
    return x.to(TDT[dtype])


# ----------------------------------------------------------------- score ----
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("G,n_split,S", [(1, 0, 1037), (4, 3, 1037), (2, 7, 600), (1, 1, 64), (1, 0, 5), (4, 64, 4100)])
def test_score_matches_oracle(dtype, G, n_split, S):
    L, B, N_kv, S_obs = 2, 2, 2, min(32, S)
    q_obs = _randn((L, B, N_kv * G, S_obs, D), dtype, 11)
    k = _randn((L, B, N_kv, S, D), dtype, 12)
    shape = thk.make_shape(L, B, N_kv * G, N_kv, D, S, S_obs, 64, 0, DT[dtype], n_split)
    got = gpu_score(shape, q_obs, k).cpu().numpy().astype(np.float64).reshape(L, B, N_kv, D)
    want = O.score(as_numpy(q_obs), as_numpy(k), dtype)
    rel = np.abs(got - want) / want
    print(f"score {dtype} G={G} split={n_split} S={S}: max rel err {rel.max():.3e}")
    assert rel.max() <= SCORE_TOL


MAGNITUDE_CASES = [
    # dtype, L, B, N_kv, S, n_split, sigma
    ("bf16", 1, 2, 3, 777, 0, 1.0),
    ("f32", 1, 2, 3, 777, 0, 1.0),
    ("bf16", 4, 2, 8, 4100, 0, 1.5),     # a layer stack in one call, several splits, ragged pieces
    ("f32", 3, 1, 5, 2049, 7, 2.0),
    ("bf16", 1, 1, 1, 5, 1, 0.0),        # shorter than one row group
    ("f32", 2, 1, 2, 33000, 0, 1.0),     # long units: fp32 chains folded into fp64 many times
]


@pytest.mark.parametrize("p", [1, 2])
@pytest.mark.parametrize("dtype,L,B,N_kv,S,n_split,sigma", MAGNITUDE_CASES)
def test_magnitude_score_matches_oracle(dtype, L, B, N_kv, S, n_split, sigma, p):
    """Eq. 1: M[n, d] = ||K[n, :, d]||_p, p = 1, 2, and the Top_T taken from it."""
    k = _randn((L, B, N_kv, S, D), dtype, 13 + S, sigma)
    shape = thk.make_shape(L, B, N_kv, N_kv, D, S, 1, 64, 0, DT[dtype], n_split)
    U = L * B * N_kv
    score = torch.empty(U, D, dtype=torch.float32, device="cuda")
    ws = ws_tensor(thk.thk_workspace_bytes(shape, thk.THK_OP_SCORE))
    thk.thk_score_magnitude(shape, k, p, score, ws)
    torch.cuda.synchronize()
    want = O.score_magnitude(as_numpy(k), dtype, p).reshape(U, D)
    rel = np.abs(score.cpu().numpy().astype(np.float64) - want) / want
    assert rel.max() <= SCORE_TOL
    # I = Top_T(M, T): the list from the GPU's scores against the oracle's, up to exact-tolerance ties
    idx = gpu_select(shape, score).cpu().numpy()
    check_idx_with_tie_rule(idx, O.select_topk(want, 64), want, 64)


# ---------------------------------------------------------------- select ----
@pytest.mark.parametrize("T", [1, 2, 51, 63, 64, 65, 76, 127, 128])
def test_select_bit_exact_on_same_scores(T):
    """Both sides decide on the same fp32 scores: no tolerance."""
    U = 70
    g = torch.Generator(device="cuda"); g.manual_seed(100 + T)
    score = torch.randn(U, D, generator=g, device="cuda").abs()
    score[3] = score[3].round(decimals=1)      # many exact ties
    score[4] = 0.0                             # all equal
    score[5, ::2] = score[5, 1::2]             # duplicated pairs
    score[6] = torch.arange(D, device="cuda").float()        # ascending
    score[7] = torch.arange(D, 0, -1, device="cuda").float()  # descending
    shape = thk.make_shape(1, 1, U, U, D, 1, 1, T, 0, thk.THK_F32, 0)
    got = gpu_select(shape, score).cpu().numpy()
    want = O.select_topk(score.cpu().numpy().astype(np.float64), T)
    np.testing.assert_array_equal(got, want)


# --------------------------------------------------------------- compact ----
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("S,T,ld", [(1024, 64, 0), (1056, 76, 0), (2048 + 32, 51, 0), (1037, 51, 0), (1037, 76, 80),
                                     (520, 128, 0), (16, 1, 0), (3, 7, 0), (4096, 89, 0), (8, 51, 0),
                                     # padded rows, pitches that are and are not multiples of 16 bytes
                                     (300, 51, 56), (300, 51, 53), (64, 7, 8), (555, 100, 128), (33, 3, 8), (700, 89, 92)])
def test_compact_bit_exact(dtype, S, T, ld):
    L, B, N_kv = 1, 2, 3
    k = _randn((L, B, N_kv, S, D), dtype, 21)
    g = torch.Generator(device="cpu"); g.manual_seed(S + T)
    score = torch.rand(L * B * N_kv, D, generator=g).numpy().astype(np.float64)
    idx_np = O.select_topk(score, T)
    idx = torch.from_numpy(idx_np).cuda()
    shape = thk.make_shape(L, B, N_kv, N_kv, D, S, 1, T, ld, DT[dtype], 0)
    kp = gpu_compact(shape, k, idx, fill=7)            # every element of every row is written:
    want = O.compact_keys(as_numpy(k).reshape(L * B * N_kv, S, D), idx_np, dtype, ld)
    np.testing.assert_array_equal(as_numpy(kp), want)   # the padding columns as zeros


# ---------------------------------------------------------------- decode ----
def _decode_case(dtype, B, N_kv, G, S, T, ld, n_split, s_tail, cap, sigma, seed):
    N_q = N_kv * G
    q = _randn((1, B, N_q, D), dtype, seed, sigma)
    k = _randn((1, B, N_kv, S, D), dtype, seed + 1, sigma)
    v = _randn((1, B, N_kv, S, D), dtype, seed + 2, 0)
    kt = _randn((1, B, N_kv, max(cap, 1), D), dtype, seed + 3, sigma)
    vt = _randn((1, B, N_kv, max(cap, 1), D), dtype, seed + 4, 0)
    g = torch.Generator(device="cpu"); g.manual_seed(seed + 5)
    idx_np = O.select_topk(torch.rand(B * N_kv, D, generator=g).numpy().astype(np.float64), T)
    idx = torch.from_numpy(idx_np).cuda()
    shape = thk.make_shape(1, B, N_q, N_kv, D, S, 1, T, ld, DT[dtype], n_split)
    kp = gpu_compact(shape, k, idx)
    out = gpu_decode(shape, q, kp, idx, v, kt if s_tail else None, vt if s_tail else None, s_tail, cap)
    U = B * N_kv
    ref = O.decode_attn(as_numpy(q)[0], as_numpy(kp).reshape(B, N_kv, S, -1), idx_np.reshape(B, N_kv, T),
                        as_numpy(v)[0], dtype, as_numpy(kt)[0] if s_tail else None,
                        as_numpy(vt)[0] if s_tail else None, s_tail)
    err = attn_rel_err(out, ref.reshape(B * N_q, D))
    return err, out


DECODE_CASES = [
    # B N_kv G   S    T   ld split tail cap sigma
    (2, 2, 1, 1037, 64, 0, 0, 0, 0, 1.0),
    (2, 2, 1, 1037, 76, 0, 0, 0, 0, 1.0),
    (2, 2, 1, 1037, 51, 0, 0, 0, 0, 1.0),
    (1, 2, 4, 1037, 64, 0, 3, 0, 0, 1.0),
    (1, 2, 4, 2048, 76, 0, 0, 17, 64, 1.0),
    (1, 1, 8, 1500, 51, 0, 2, 64, 64, 1.0),
    (1, 1, 3, 700, 64, 0, 0, 1, 4, 1.0),
    (1, 2, 2, 900, 89, 0, 7, 5, 16, 1.0),
    (1, 2, 1, 1, 64, 0, 0, 0, 0, 1.0),
    (1, 2, 1, 1, 64, 0, 0, 1, 1, 1.0),
    (1, 2, 1, 63, 128, 0, 0, 0, 0, 1.0),
    (1, 2, 1, 65, 1, 0, 0, 0, 0, 1.0),
    (1, 2, 1, 300, 7, 0, 2, 3, 8, 1.0),
    (1, 2, 1, 1037, 76, 80, 0, 0, 0, 1.0),
    (1, 2, 1, 1037, 51, 56, 4, 9, 16, 1.0),
    (2, 3, 1, 4096, 76, 0, 0, 0, 0, 0.0),      # diffuse softmax: V accumulation dominates
    (1, 2, 4, 8192, 64, 0, 64, 0, 0, 0.0),
    (1, 2, 1, 5000, 64, 0, 0, 33, 64, 2.0),    # heavy-tailed scales: near one-hot softmax
    # four query heads per KV head: bf16 takes the matrix-core kernel when T and ld are multiples of 4
    (1, 2, 4, 1037, 76, 80, 0, 0, 0, 1.0),     # padded rows
    (1, 1, 4, 333, 128, 0, 2, 7, 16, 1.0),     # nothing pruned: the wide staging class
    (1, 2, 4, 100, 4, 0, 0, 0, 0, 1.0),        # one chunk per row
    (1, 2, 4, 97, 8, 12, 0, 16, 16, 1.0),
    (1, 1, 8, 2100, 64, 0, 5, 33, 64, 0.0),    # two groups of four heads
    (1, 2, 4, 1, 64, 0, 0, 0, 0, 1.0),
    (1, 2, 4, 1, 64, 0, 0, 1, 1, 1.0),
    (1, 2, 4, 500, 64, 66, 0, 3, 8, 1.0),      # pitch not a multiple of 4
    (1, 1, 4, 4096, 76, 0, 0, 64, 64, 2.0),
    (1, 1, 4, 200, 124, 0, 0, 2, 4, 1.0),      # 248-byte rows: 8-byte aligned only
    (1, 1, 4, 200, 124, 128, 2, 0, 0, 1.0),    # the widest padded rows: pitch D
    (1, 2, 4, 555, 64, 128, 0, 5, 8, 0.0),     # kept channels at the front of full-width rows
    # eight query heads per KV head share one block (and every key / value byte)
    (1, 1, 16, 700, 76, 0, 0, 3, 8, 1.0),      # two blocks of eight heads
    (1, 2, 12, 400, 64, 0, 0, 0, 0, 1.0),      # 12 heads: three blocks of four
    (1, 1, 8, 333, 124, 128, 2, 5, 16, 1.0),   # the widest staging class
    (2, 2, 8, 4133, 76, 0, 0, 40, 64, 0.0),
    # head counts that do not fill the blocks' slots: the last block of a unit leaves some empty
    (1, 2, 3, 900, 64, 0, 2, 5, 16, 1.0),      # bf16: 3 of 4 matrix-core slots; f32: 3 of 4 general slots
    (1, 2, 5, 1300, 76, 0, 0, 0, 0, 1.0),      # 5 of 8
    (1, 1, 7, 650, 128, 0, 3, 17, 32, 0.0),    # 7 of 8, the wide staging class
    (1, 1, 9, 500, 64, 0, 0, 0, 0, 1.0),       # 8 + 1
    (1, 2, 6, 800, 51, 0, 2, 9, 16, 1.0),      # T not a multiple of 4
    (1, 2, 5, 300, 51, 56, 0, 0, 0, 1.0),
]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("case", DECODE_CASES, ids=lambda c: "-".join(map(str, c)))
def test_decode_matches_oracle(dtype, case, decode_merge):
    B, N_kv, G, S, T, ld, n_split, s_tail, cap, sigma = case
    err, _ = _decode_case(dtype, B, N_kv, G, S, T, ld, n_split, s_tail, cap, sigma, 1000 + S + T)
    print(f"decode {dtype} {case}: max rel err {err.max():.3e}")
    assert err.max() <= ATTN_TOL[dtype]


@pytest.mark.parametrize("case", [c for c in DECODE_CASES if c[2] >= 3], ids=lambda c: "-".join(map(str, c)))
def test_decode_general_kernel_on_grouped_heads(case, thk_env, decode_merge):
    """THK_DECODE_MFMA=0 keeps bf16 shapes with three or more query heads per KV head on the general kernel."""
    thk_env.setenv("THK_DECODE_MFMA", "0")
    B, N_kv, G, S, T, ld, n_split, s_tail, cap, sigma = case
    err, out0 = _decode_case("bf16", B, N_kv, G, S, T, ld, n_split, s_tail, cap, sigma, 1000 + S + T)
    assert err.max() <= ATTN_TOL["bf16"]
    thk_env.setenv("THK_DECODE_MFMA", "1")
    err1, out1 = _decode_case("bf16", B, N_kv, G, S, T, ld, n_split, s_tail, cap, sigma, 1000 + S + T)
    print(f"decode bf16 {case}: max rel err general {err.max():.3e}, matrix cores {err1.max():.3e}")
    assert err1.max() <= ATTN_TOL["bf16"]


@pytest.mark.parametrize("G,T,ld", [(4, 51, 52), (8, 89, 92), (3, 1, 4), (5, 38, 40), (8, 127, 128)])
def test_decode_ignores_whatever_sits_in_the_row_padding(G, T, ld):
    """Rows of T kept channels padded to a multiple of 4 elements run on the matrix-core kernel, which
    reads whole 4-element chunks: what the padding holds (here NaN) must not reach the logits."""
    B, N_kv, S, s_tail, cap = 1, 2, 1234, 7, 16
    N_q = N_kv * G
    q = _randn((1, B, N_q, D), "bf16", 31, 1.0)
    k = _randn((1, B, N_kv, S, D), "bf16", 32, 1.0)
    v = _randn((1, B, N_kv, S, D), "bf16", 33, 0)
    kt = _randn((1, B, N_kv, cap, D), "bf16", 34, 1.0)
    vt = _randn((1, B, N_kv, cap, D), "bf16", 35, 0)
    g = torch.Generator(device="cpu"); g.manual_seed(36)
    idx_np = O.select_topk(torch.rand(B * N_kv, D, generator=g).numpy().astype(np.float64), T)
    idx = torch.from_numpy(idx_np).cuda()
    shape = thk.make_shape(1, B, N_q, N_kv, D, S, 1, T, ld, thk.THK_BF16, 0)
    assert thk.thk_decode_on_matrix_cores(shape) == 1
    kp = gpu_compact(shape, k, idx)
    kp[:, :, T:] = float("nan")
    out = gpu_decode(shape, q, kp, idx, v, kt, vt, s_tail, cap)
    ref = O.decode_attn(as_numpy(q)[0], as_numpy(kp).reshape(B, N_kv, S, -1), idx_np.reshape(B, N_kv, T),
                        as_numpy(v)[0], "bf16", as_numpy(kt)[0], as_numpy(vt)[0], s_tail)
    err = attn_rel_err(out, ref.reshape(B * N_q, D))
    assert np.isfinite(out.float().cpu().numpy()).all()
    assert err.max() <= ATTN_TOL["bf16"]


@pytest.mark.parametrize("G", [4, 7])
@pytest.mark.parametrize("T,ld", [(1, 0), (2, 0), (3, 0), (4, 5), (5, 0), (7, 0), (8, 9), (9, 10), (50, 51), (51, 0), (62, 0),
                                  (66, 0), (77, 0), (79, 0), (81, 0), (126, 0), (127, 0), (51, 127)])
def test_decode_matrix_cores_any_row_pitch(T, ld, G):
    """Key rows that are not a multiple of 4 elements apart: rows start on a word or in the middle of
    one, a row has fewer chunks than halves (T < 8), an odd chunk, a partial chunk, both or
    neither, and the rows of a ragged last tile and of the tail follow."""
    assert thk.thk_decode_on_matrix_cores(thk.make_shape(1, 1, 3 * G, 3, D, 161, 1, T, ld, thk.THK_BF16, 0)) == 1
    err, out = _decode_case("bf16", 1, 3, G, 161, T, ld, 0, 19, 32, 1.0, 4000 + 7 * T + ld)
    assert np.isfinite(out.float().cpu().numpy()).all()
    assert err.max() <= ATTN_TOL["bf16"]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_decode_split_invariance_and_determinism(dtype, decode_merge):
    outs = {}
    for n_split in (1, 2, 7, 64):
        err, out = _decode_case(dtype, 1, 2, 4, 8192 + 100, 64, 0, n_split, 11, 16, 1.0, 77)
        assert err.max() <= ATTN_TOL[dtype]
        _, out2 = _decode_case(dtype, 1, 2, 4, 8192 + 100, 64, 0, n_split, 11, 16, 1.0, 77)
        assert torch.equal(out, out2), "two runs must be bit-identical (no atomics)"
        outs[n_split] = out.float()
    ref = outs[1]
    for n_split, o in outs.items():
        rel = ((o - ref).abs().amax(-1) / ref.abs().amax(-1)).max().item()
        assert rel <= ATTN_TOL[dtype], f"n_split={n_split} deviates by {rel}"


@pytest.mark.parametrize("dtype,G,S,tail", [("bf16", 1, 1000, 0), ("bf16", 4, 70000, 9), ("f32", 2, 300, 3)])
def test_decode_with_the_largest_split_count(dtype, G, S, tail):
    """n_split = 4096, the most the interface takes: nearly every piece is empty (64 rows per piece
    at least, so S = 70000 fills 1094 of them and S = 300 five); empty pieces must carry a weight
    of zero into the merge, and the tail tiles go to pieces that have no pruned rows at all."""
    err, out = _decode_case(dtype, 1, 2, G, S, 64, 0, 4096, tail, 16, 1.0, 123)
    assert np.isfinite(out.float().cpu().numpy()).all()
    assert err.max() <= ATTN_TOL[dtype]
    _, out1 = _decode_case(dtype, 1, 2, G, S, 64, 0, 1, tail, 16, 1.0, 123)
    rel = ((out.float() - out1.float()).abs().amax(-1) / out1.float().abs().amax(-1)).max().item()
    assert rel <= ATTN_TOL[dtype]


# ----------------------------------------------------------------- prune ----
PRUNE_CASES = [("bf16", 1, 2048, 76, 1.5), ("bf16", 4, 4096 + 64, 64, 1.0), ("f32", 1, 1037, 64, 1.0),
               ("bf16", 1, 1024, 51, 2.0), ("f32", 2, 2048, 64, 1.0), ("bf16", 1, 40, 64, 1.0)]


@pytest.mark.parametrize("levels", [1, 2])
def test_prune_fused_repeated_calls_on_one_workspace(levels, thk_env, prune_launch):
    """The one-launch form hands sums and index lists from block to block through the
    workspace (one level: the last block's list to the blocks that wait; two levels: the group
    vectors to every block of the unit).  Calls that alternate between two inputs on the SAME
    workspace leave the other input's words behind each time: a block that picked up stale
    words (or words that had not fully arrived) would compact the wrong channels.  Checked
    on the GPU against a plain gather with the index list the call returned, and against the
    oracle's list for the first call of each input."""
    thk_env.setenv("THK_PRUNE_PATH", "fused")
    if levels == 1:
        L, B, N, S, S_obs, T = 4, 4, 16, 4096, 32, 76
    else:                                          # 102 blocks of 128 rows per unit
        thk_env.setenv("THK_PRUNE_BLOCK_ROWS", "128")
        L, B, N, S, S_obs, T = 1, 3, 4, 13008, 32, 64
    U = L * B * N
    shape = thk.make_shape(L, B, N, N, D, S, S_obs, T, 0, thk.THK_BF16, 0)
    assert thk.thk_prune_is_fused(shape) == 2      # the form that keeps the rows on chip
    inputs = [(_randn((L, B, N, S_obs, D), "bf16", 71 + i, 1.0), _randn((L, B, N, S, D), "bf16", 81 + i, 1.0))
              for i in range(2)]
    ws = ws_tensor(thk.thk_workspace_bytes(shape, thk.THK_OP_PRUNE))
    ws.fill_(0xA5)
    score = torch.empty(U, D, dtype=torch.float32, device="cuda")
    idx = torch.empty(U, T, dtype=torch.int16, device="cuda")
    kp = torch.empty(U, S, T, dtype=torch.bfloat16, device="cuda")
    first_idx = {}
    for rep in range(8):
        q_obs, k = inputs[rep % 2]
        kp.fill_(-7.0)
        thk.thk_prune(shape, q_obs, k, score, idx, kp, ws)
        torch.cuda.synchronize()
        want = torch.gather(k.reshape(U, S, D), 2, idx.to(torch.int64)[:, None, :].expand(U, S, T))
        assert torch.equal(kp.view(torch.int16), want.view(torch.int16)), f"call {rep}"
        if rep < 2:
            first_idx[rep] = idx.clone()
            o_sc = O.score(as_numpy(q_obs), as_numpy(k), "bf16").reshape(U, D)
            check_idx_with_tie_rule(idx.cpu().numpy(), O.select_topk(o_sc, T), o_sc, T)
        else:
            assert torch.equal(idx, first_idx[rep % 2]), f"call {rep}"
    assert not torch.equal(first_idx[0], first_idx[1])


@pytest.mark.parametrize("levels", [1, 2])
@pytest.mark.parametrize("delay_us", [30, 200])
def test_prune_single_launch_with_a_late_prologue(levels, delay_us, thk_env):
    """The single-launch prune initialises its hand-off state inside the launch: a prologue block
    per unit clears it and then tags the unit's arrival counters with the call's nonce; a row
    block that arrives earlier finds a foreign tag, waits for the right one and arrives again.
    Here the prologue is held back from the host (THK_PRUNE_PROLOGUE_DELAY_US) so that EVERY row
    block arrives first -- on a workspace full of garbage, on the state the previous call left,
    and with the wait for the index list switched off as well (spin limit 0: the blocks give up
    and the unit's finisher compacts their rows).  Every kernel exits normally; results as ever."""
    thk_env.setenv("THK_PRUNE_LAUNCH", "solo")
    thk_env.setenv("THK_PRUNE_PROLOGUE_DELAY_US", str(delay_us))
    if levels == 1:
        L, B, N, G, S, S_obs, T = 2, 2, 4, 2, 3000, 32, 76
    else:                                          # 102 blocks of 128 rows per unit: two levels of sums
        thk_env.setenv("THK_PRUNE_BLOCK_ROWS", "128")
        L, B, N, G, S, S_obs, T = 1, 2, 2, 1, 13008, 32, 64
    U = L * B * N
    shape = thk.make_shape(L, B, N * G, N, D, S, S_obs, T, 0, thk.THK_BF16, 0)
    assert thk.thk_prune_launches(shape) == 1
    ws = ws_tensor(thk.thk_workspace_bytes(shape, thk.THK_OP_PRUNE))
    score = torch.empty(U, D, dtype=torch.float32, device="cuda")
    idx = torch.empty(U, T, dtype=torch.int16, device="cuda")
    kp = torch.empty(U, S, T, dtype=torch.bfloat16, device="cuda")
    for rep, (fill, spin) in enumerate([(0xA5, None), (None, None), (0xFF, "0"), (None, "0"), (0x00, None)]):
        if fill is not None:
            ws.fill_(fill)
        if spin is not None:
            thk_env.setenv("THK_PRUNE_SPIN_LIMIT", spin)
        q_obs = _randn((L, B, N * G, S_obs, D), "bf16", 171 + rep, 1.0)
        k = _randn((L, B, N, S, D), "bf16", 181 + rep, 1.0)
        kp.fill_(-7.0)
        thk.thk_prune(shape, q_obs, k, score, idx, kp, ws)
        torch.cuda.synchronize()
        o_sc, o_idx, _ = oracle_prune(q_obs, k, "bf16", T)
        rel = np.abs(score.cpu().numpy().astype(np.float64) - o_sc.reshape(U, D)) / o_sc.reshape(U, D)
        assert rel.max() <= SCORE_TOL, f"call {rep}"
        check_idx_with_tie_rule(idx.cpu().numpy(), o_idx, o_sc, T)
        want = O.compact_keys(as_numpy(k).reshape(U, S, D), idx.cpu().numpy(), "bf16")
        np.testing.assert_array_equal(as_numpy(kp), want, err_msg=f"call {rep}")


@pytest.mark.parametrize("dtype,G,S,T,ld,block_rows", [("bf16", 1, 4096, 76, 80, ""), ("bf16", 4, 3001, 51, 56, "128"),
                                                       ("f32", 1, 1037, 51, 52, ""), ("bf16", 1, 2048, 76, 88, "64"),
                                                       ("bf16", 2, 777, 100, 104, "32"), ("bf16", 1, 1500, 76, 77, "")])
def test_prune_into_padded_rows(dtype, G, S, T, ld, block_rows, thk_env, prune_launch):
    """K_pruned rows with padding behind them, whatever the pitch: the one-launch prune serves them
    and the padding columns are written as zeros."""
    if block_rows:
        thk_env.setenv("THK_PRUNE_BLOCK_ROWS", block_rows)
    L, B, N_kv, S_obs = 1, 2, 3, 32
    U = L * B * N_kv
    q_obs = _randn((L, B, N_kv * G, S_obs, D), dtype, 61, 1.0)
    k = _randn((L, B, N_kv, S, D), dtype, 62, 1.0)
    shape = thk.make_shape(L, B, N_kv * G, N_kv, D, S, S_obs, T, ld, DT[dtype], 0)
    assert thk.thk_prune_is_fused(shape) != 0
    score = torch.empty(U, D, dtype=torch.float32, device="cuda")
    idx = torch.empty(U, T, dtype=torch.int16, device="cuda")
    kp = torch.full((U, S, ld), 7, dtype=k.dtype, device="cuda")
    thk.thk_prune(shape, q_obs, k, score, idx, kp, ws_tensor(thk.thk_workspace_bytes(shape, thk.THK_OP_PRUNE)))
    torch.cuda.synchronize()
    o_sc, o_idx, _ = oracle_prune(q_obs, k, dtype, T, ld)
    check_idx_with_tie_rule(idx.cpu().numpy(), o_idx, o_sc.reshape(U, D), T)
    want = O.compact_keys(as_numpy(k).reshape(U, S, D), idx.cpu().numpy(), dtype, ld)   # zeros in the padding
    np.testing.assert_array_equal(as_numpy(kp), want)


@pytest.mark.parametrize("spin_limit", [None, 0])
@pytest.mark.parametrize("block_rows,S", [(128, 13008), (64, 13008), (128, 40016)])
def test_prune_two_level_arrival(block_rows, S, spin_limit, thk_env, prune_launch):
    """Units of more than 64 row blocks: the blocks arrive group by group, the last block of a
    group publishes the group's sums, and every block makes the index list from the group sums
    (102 blocks of 128 rows held on chip; 204 blocks of 64 rows read twice).  With the wait
    switched off from the host, blocks that find a group vector missing leave their rows, and
    possibly the caller's copy of the list, to the repair kernel."""
    thk_env.setenv("THK_PRUNE_PATH", "fused")
    thk_env.setenv("THK_PRUNE_BLOCK_ROWS", str(block_rows))
    if spin_limit is not None:
        thk_env.setenv("THK_PRUNE_SPIN_LIMIT", str(spin_limit))
    L, B, N_kv, G, S_obs, T = 1, 2, 2, 2, 32, 64       # S = 40016: 313 blocks per unit, groups of 20
    q_obs = _randn((L, B, N_kv * G, S_obs, D), "bf16", 41, 1.0)
    k = _randn((L, B, N_kv, S, D), "bf16", 42, 1.0)
    shape = thk.make_shape(L, B, N_kv * G, N_kv, D, S, S_obs, T, 0, thk.THK_BF16, 0)
    assert thk.thk_prune_is_fused(shape) == (2 if block_rows == 128 else 1)
    score, idx, kp = gpu_prune(shape, q_obs, k)
    o_sc, o_idx, o_kp = oracle_prune(q_obs, k, "bf16", T)
    U = L * B * N_kv
    rel = np.abs(score.cpu().numpy().astype(np.float64) - o_sc.reshape(U, D)) / o_sc.reshape(U, D)
    assert rel.max() <= SCORE_TOL
    check_idx_with_tie_rule(idx.cpu().numpy(), o_idx, o_sc, T)
    np.testing.assert_array_equal(as_numpy(kp), O.compact_keys(as_numpy(k).reshape(U, S, D), idx.cpu().numpy(), "bf16"))


@pytest.mark.parametrize("dtype,block_rows,n_blocks,short", [
    ("bf16", 128, 1, 127), ("bf16", 128, 2, 1), ("bf16", 128, 47, 96), ("bf16", 128, 48, 0), ("bf16", 128, 49, 33),
    ("bf16", 128, 64, 127), ("bf16", 128, 65, 31), ("bf16", 256, 33, 255), ("bf16", 512, 17, 129), ("f32", 128, 49, 65),
    ("f32", 256, 18, 1)])
def test_prune_single_launch_block_counts(dtype, block_rows, n_blocks, short, thk_env):
    """The single-launch prune at the edges of its batches and tiles: the column sums of a unit's
    blocks are merged 8, 16 or 24 vectors per thread group and batch (one block; exactly two groups
    of 24; one more; the last one-level and the first two-level count), and the last block lacks
    `short` rows (none; whole 32-row tiles; all but one row)."""
    thk_env.setenv("THK_PRUNE_LAUNCH", "solo")
    thk_env.setenv("THK_PRUNE_BLOCK_ROWS", str(block_rows))
    L, B, N_kv, G, S_obs, T = 1, 1, 3, 2, 8, 77
    S = block_rows * n_blocks - short
    U = L * B * N_kv
    S_obs = min(S_obs, S)
    q_obs = _randn((L, B, N_kv * G, S_obs, D), dtype, 301, 1.0)
    k = _randn((L, B, N_kv, S, D), dtype, 302, 1.0)
    shape = thk.make_shape(L, B, N_kv * G, N_kv, D, S, S_obs, T, 0, DT[dtype], 0)
    assert thk.thk_prune_launches(shape) == 1
    for _ in range(2):      # the second call finds the first one's workspace state
        score, idx, kp = gpu_prune(shape, q_obs, k)
        o_sc, o_idx, _ = oracle_prune(q_obs, k, dtype, T)
        rel = np.abs(score.cpu().numpy().astype(np.float64) - o_sc.reshape(U, D)) / o_sc.reshape(U, D)
        assert rel.max() <= SCORE_TOL
        check_idx_with_tie_rule(idx.cpu().numpy(), o_idx, o_sc, T)
        np.testing.assert_array_equal(as_numpy(kp), O.compact_keys(as_numpy(k).reshape(U, S, D), idx.cpu().numpy(), dtype))


@pytest.mark.parametrize("rest", [1, 33, -31])
@pytest.mark.parametrize("dtype,U,NB", [("bf16", 16, 49), ("bf16", 11, 70), ("f32", 16, 33), ("f32", 8, 65)])
def test_prune_single_launch_of_more_than_one_round(dtype, U, NB, rest, thk_env):
    """Single launches of a few blocks more than are resident at once (768, fp32 512), with one level of sums and with two
    (more than 64 blocks a unit): the last block of every unit has one row, a tile and a row, or all but 31; rows of one element to
    128, dense and padded, the last rows left alone or not; behind the list, and with every block but a unit's last
    resigning while rows of the next round are on their way."""
    thk_env.setenv("THK_PRUNE_LAUNCH", "solo")
    block_rows = 512 if dtype == "bf16" else 256
    S, G, S_obs = block_rows * (NB if rest < 0 else NB - 1) + rest, 2, 8
    assert U * NB > (768 if dtype == "bf16" else 512)
    q_obs = _randn((1, 1, U * G, S_obs, D), dtype, 311 + rest, 1.0)
    k = _randn((1, 1, U, S, D), dtype, 312 + rest, 1.0)
    kd = k.reshape(U, S, D)
    norms = torch.stack([x.double().square().sum(0).sqrt() for x in kd])
    want = (norms * q_obs.reshape(U, G, S_obs, D).double().square().sum(2).sqrt().sum(1)).cpu().numpy()
    for T, ld, recent in [(1, 0, 0), (7, 0, 33), (51, 0, 0), (128, 0, 1), (7, 12, 0), (1, 5, 32), (51, 56, 40), (12, 0, 0)]:
        shape = thk.make_shape(1, 1, U * G, U, D, S, S_obs, T, ld, DT[dtype], 0, recent)
        assert thk.thk_prune_launches(shape) == 1
        rows, n = S - recent, U * (S - recent) * (ld or T)
        score, idx = torch.empty(U, D, device="cuda"), torch.empty(U, T, dtype=torch.int16, device="cuda")
        ws = ws_tensor(thk.thk_workspace_bytes(shape, thk.THK_OP_PRUNE))
        for spin in (None, "0"):
            if spin is None:
                thk_env.delenv("THK_PRUNE_SPIN_LIMIT", raising=False)
            else:
                thk_env.setenv("THK_PRUNE_SPIN_LIMIT", spin)
            kp = torch.full((n + 64,), 3.0, dtype=k.dtype, device="cuda")   # what lies behind the last row stays
            thk.thk_prune(shape, q_obs, k, score, idx, kp, ws)
            torch.cuda.synchronize()
            where = f"T={T} ld={ld} recent={recent} spin={spin}"
            assert np.abs(score.cpu().numpy() / want - 1).max() <= SCORE_TOL, where
            check_idx_with_tie_rule(idx.cpu().numpy(), O.select_topk(want, T), want, T)
            got = kp[:n].reshape(U, rows, -1)
            for u in range(U):
                assert torch.equal(got[u, :, :T], kd[u, :rows, idx[u].long()]), (where, u)
            assert (got[..., T:] == 0).all() and (kp[n:] == 3).all(), where


@pytest.mark.parametrize("path", ["fused", "fused-small-blocks", "fused-no-wait", "hold-128", "hold-256", "hold-512",
                                  "hold-256-no-wait", "reread-256", "staged", "staged-groups"])
@pytest.mark.parametrize("dtype,G,S,T,sigma", PRUNE_CASES)
def test_prune_pipeline_matches_oracle(dtype, G, S, T, sigma, path, thk_env, prune_launch):
    """thk_prune in its one-launch form (default row blocks, 32-row blocks, and with
    the wait for the index list switched off from the host so that the repair
    kernel does every compaction) and in its staged form (one group, many groups)."""
    if prune_launch == "solo" and not (path.startswith("hold") or path in ("fused", "fused-no-wait")):
        pytest.skip("the single-launch form exists only where the rows are held on chip")
    if path.startswith("fused") or path.startswith("hold"):
        thk_env.setenv("THK_PRUNE_PATH", "fused")
    if path.startswith("hold"):      # row blocks that stay in registers between score and compaction
        thk_env.setenv("THK_PRUNE_BLOCK_ROWS", path.split("-")[1])
    if path == "hold-256-no-wait":
        thk_env.setenv("THK_PRUNE_SPIN_LIMIT", "0")
    if path == "reread-256":         # the same blocking with the rows read twice
        thk_env.setenv("THK_PRUNE_PATH", "reread")
        thk_env.setenv("THK_PRUNE_BLOCK_ROWS", "256")
    if path == "fused-small-blocks":
        thk_env.setenv("THK_PRUNE_BLOCK_ROWS", "32")
    if path == "fused-no-wait":
        thk_env.setenv("THK_PRUNE_SPIN_LIMIT", "0")
    if path.startswith("staged"):
        thk_env.setenv("THK_PRUNE_PATH", "staged")
    if path == "staged-groups":
        thk_env.setenv("THK_PRUNE_GROUP_MIB", "1")     # several groups, some starting mid-batch
    L, B, N_kv, S_obs = 2, 2, 3, min(32, S)
    q_obs = _randn((L, B, N_kv * G, S_obs, D), dtype, 31, sigma)
    k = _randn((L, B, N_kv, S, D), dtype, 32, sigma)
    shape = thk.make_shape(L, B, N_kv * G, N_kv, D, S, S_obs, T, 0, DT[dtype], 0)
    score, idx, kp = gpu_prune(shape, q_obs, k)
    o_sc, o_idx, o_kp = oracle_prune(q_obs, k, dtype, T)
    U = L * B * N_kv
    rel = np.abs(score.cpu().numpy().astype(np.float64) - o_sc.reshape(U, D)) / o_sc.reshape(U, D)
    assert rel.max() <= SCORE_TOL
    differing = check_idx_with_tie_rule(idx.cpu().numpy(), o_idx, o_sc, T)
    kp_np, o_kp = as_numpy(kp), o_kp.reshape(U, S, T)
    same = [u for u in range(U) if u not in differing]
    np.testing.assert_array_equal(kp_np[same], o_kp[same])
    # the compacted keys are exactly the gather with the index list the call itself produced
    np.testing.assert_array_equal(kp_np, O.compact_keys(as_numpy(k).reshape(U, S, D), idx.cpu().numpy(), dtype))
    # the separate entry points: same bits as the staged call; the one-launch form sums the
    # partial column sums in another order, so its scores may differ in the last float bit
    sc2 = gpu_score(shape, q_obs, k)
    idx2 = gpu_select(shape, sc2)
    kp2 = gpu_compact(shape, k, idx2)
    if path.startswith("staged"):
        assert torch.equal(sc2, score) and torch.equal(idx2, idx) and torch.equal(kp2, kp)
    else:
        assert ((sc2 - score).abs() <= 2.4e-7 * score.abs()).all()
    # a second call on the same workspace gives the same bits (counters are reset per call)
    score_b, idx_b, kp_b = gpu_prune(shape, q_obs, k)
    assert torch.equal(score_b, score) and torch.equal(idx_b, idx) and torch.equal(kp_b, kp)


@pytest.mark.parametrize("pattern", ["pairs", "all-equal", "blocks-of-16", "half-zero"])
@pytest.mark.parametrize("T", [1, 2, 51, 64, 65, 127, 128])
def test_prune_breaks_exact_ties_by_channel_number(pattern, T, prune_launch):
    """Channels that are copies of each other score the same to the last bit (on the GPU and in the
    oracle alike), so Top_T has to fall back on its tie rule -- the lower channel number wins
    (Sec. 3.2's Top_T is silent on ties; the stable order is this build's reading).  The whole
    prune call must then give exactly the oracle's list: with pairs of copies, with 16 copies
    of each of 8 columns (the T-th place falls inside a run of equal scores for most T), and with
    128 equal channels (the list is 0 .. T-1); and with 64 channels that are zero everywhere
    (scores of exactly 0, the smallest key there is: for T > 64 the list ends with the lowest zeros)."""
    L, B, N_kv, G, S, S_obs = 1, 2, 3, 2, 777, 32
    src = {"pairs": torch.arange(D) // 2 * 2, "all-equal": torch.zeros(D, dtype=torch.long),
           "blocks-of-16": torch.arange(D) % 8, "half-zero": torch.arange(D)}[pattern].cuda()
    q_obs = _randn((L, B, N_kv * G, S_obs, D), "bf16", 41)[..., src].contiguous()
    k = _randn((L, B, N_kv, S, D), "bf16", 42)[..., src].contiguous()
    if pattern == "half-zero":      # every third and every fourth channel all zero: 64 scores of exactly +0
        k[..., (torch.arange(D) % 4 >= 2).cuda()] = 0
    shape = thk.make_shape(L, B, N_kv * G, N_kv, D, S, S_obs, T, 0, thk.THK_BF16, 0)
    score, idx, kp = gpu_prune(shape, q_obs, k)
    o_sc, o_idx, o_kp = oracle_prune(q_obs, k, "bf16", T)
    U = L * B * N_kv
    sc = score.cpu().numpy()
    assert (sc == sc[:, src.cpu().numpy()]).all(), "copies of a channel must score the same bits"
    np.testing.assert_array_equal(idx.cpu().numpy(), o_idx.reshape(U, T))
    np.testing.assert_array_equal(as_numpy(kp), o_kp.reshape(U, S, T))


def test_tail_append():
    L, B, N_kv, cap = 1, 3, 5, 8
    shape = thk.make_shape(L, B, N_kv, N_kv, D, 16, 1, 64, 0, thk.THK_BF16, 0)
    kt = torch.zeros(L * B * N_kv, cap, D, dtype=torch.bfloat16, device="cuda"); vt = torch.zeros_like(kt)
    news = []
    for j in range(cap):
        kn = _randn((L * B * N_kv, D), "bf16", 50 + j); vn = _randn((L * B * N_kv, D), "bf16", 90 + j)
        thk.thk_tail_append(shape, kn, vn, kt, vt, j, cap)
        news.append((kn, vn))
    torch.cuda.synchronize()
    for j, (kn, vn) in enumerate(news):
        assert torch.equal(kt[:, j], kn) and torch.equal(vt[:, j], vn)
    with pytest.raises(thk.ThkError):
        thk.thk_tail_append(shape, news[0][0], news[0][1], kt, vt, cap, cap)


def test_device_is_the_one_the_kernels_are_written_for():
    """gfx950: 256 compute units, 64-wide wavefronts, 160 KB of LDS per workgroup at most."""
    p = torch.cuda.get_device_properties(0)
    assert p.gcnArchName.startswith("gfx950")
    assert p.multi_processor_count == 256 and p.warp_size == 64
    assert p.shared_memory_per_block == 160 * 1024
    assert p.total_memory >= 256 * 2**30


@pytest.mark.parametrize("dtype,G,n_split,S", [("bf16", 9, 1, 300), ("bf16", 17, 3, 500), ("bf16", 24, 8, 1100), ("f32", 5, 1, 300),
                                               ("f32", 9, 5, 700), ("f32", 12, 16, 2100)])
def test_decode_several_head_groups(dtype, G, n_split, S, decode_merge):
    """More heads per KV head than a block serves: the grid is laid out in eights and rounded up (numbers of
    (unit, piece) pairs on both sides of a multiple of 8), every pair and group is served once."""
    T, s_tail = 51, 5
    for units in (1, 3, 8):
        g = torch.Generator(device="cuda"); g.manual_seed(units * 100 + G)
        rnd = lambda *d: torch.randn(*d, generator=g, device="cuda").to(TDT[dtype])
        q, kp, v = rnd(1, units * G, 128), rnd(1, units, S, T), rnd(1, units, S, 128)
        kt, vt = rnd(1, units, 16, 128), rnd(1, units, 16, 128)
        idx = torch.rand(1, units, 128, generator=g, device="cuda").argsort(-1)[..., :T].sort(-1).values.to(torch.int16).contiguous()
        out = torch.full_like(q, float("nan"))
        shape = thk.make_shape(1, 1, units * G, units, 128, S, 1, T, 0, DT[dtype], n_split)
        ws = ws_tensor(thk.thk_workspace_bytes(shape, thk.THK_OP_DECODE))
        thk.thk_decode_attn(shape, q, kp, idx, v, kt, vt, s_tail, 16, out, ws)
        qd, kd, vd = q.double()[0].view(units, G, 128), kp.double()[0], v.double()[0]
        qk = qd.gather(2, idx.long()[0][:, None].expand(units, G, T))
        logits = torch.cat([(qk[:, :, None] * kd[:, None]).sum(-1), (qd[:, :, None] * kt.double()[0, :, None, :s_tail]).sum(-1)], -1)
        p = torch.softmax(logits / 128 ** 0.5, -1)
        allv = torch.cat([vd, vt.double()[0, :, :s_tail]], 1)
        ref = torch.stack([p[u] @ allv[u] for u in range(units)]).view(1, units * G, 128)
        assert attn_rel_err(out, ref[0].cpu().numpy()).max() <= ATTN_TOL[dtype], units


@pytest.mark.parametrize("dtype,B,N_q,N_kv,T,S", [
    ("bf16", 3, 32, 32, 76, 3264), ("bf16", 3, 28, 4, 64, 8000), ("bf16", 17, 32, 8, 51, 4928), ("f32", 1, 32, 32, 64, 4032)])
def test_decode_in_the_workspace_of_a_longer_sequence(dtype, B, N_q, N_kv, T, S):
    """A workspace asked for at the final length can hold fewer pieces than a shorter length would take (here: half
    as many): the call is cut into those, writes nothing behind the workspace, and gives the result of the
    full-size one."""
    mk = lambda n: thk.make_shape(1, B, N_q, N_kv, 128, S, 1, T, 0, DT[dtype], n)
    shape, pieces = mk(0), thk.thk_default_split(mk(0), thk.THK_OP_DECODE)
    assert pieces >= 4
    need, held = (thk.thk_workspace_bytes(mk(n), thk.THK_OP_DECODE) for n in (pieces, pieces // 2))
    g = torch.Generator(device="cuda"); g.manual_seed(S + B)
    rnd = lambda *d: torch.randn(*d, generator=g, device="cuda").to(TDT[dtype])
    q, kp, v = rnd(B, N_q, 128), rnd(B, N_kv, S, T), rnd(B, N_kv, S, 128)
    kt, vt = rnd(B, N_kv, 16, 128), rnd(B, N_kv, 16, 128)
    idx = torch.rand(B, N_kv, 128, generator=g, device="cuda").argsort(-1)[..., :T].sort(-1).values.to(torch.int16).contiguous()
    outs = []
    for nbytes in (need, held):
        ws = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        out = torch.full_like(q, float("nan"))
        thk.thk_decode_attn(shape, q, kp, idx, v, kt, vt, 5, 16, out, (ws, nbytes))
        torch.cuda.synchronize()
        assert (ws[nbytes:] == 0xA5).all()
        outs.append(out)
    assert attn_rel_err(outs[1], outs[0].double().cpu().numpy()).max() <= ATTN_TOL[dtype]


@pytest.mark.parametrize("G", [4, 7])
@pytest.mark.parametrize("T,ld", [(51, 0), (70, 0), (127, 0), (51, 53)])
@pytest.mark.parametrize("second_row", ["pruned", "tail", "pruned values"])
def test_decode_probabilities_keep_24_bits_at_any_row_pitch(second_row, T, ld, G):
    """Two rows with nearly equal logits and opposite values: the output is the difference of the two
    probabilities, about 2^-13 of them, so what the kernel drops of a probability shows.  Key rows that are
    not a multiple of 4 elements apart (T = 128: the narrowest such pitch, T - 1 kept) are to keep all
    24 bits.  Bound per element: the bf16 rounding of the result, 2^-8 |out|, and 2^-20 of sum(p |v|) for
    fp32 logits (a few units of 2^-24 of at most 8 in the log2 domain) and an exp2 of one unit."""
    U, pitch = 64, ld or T
    g = torch.Generator(device="cuda"); g.manual_seed(T + G)
    rnd = lambda *d: torch.randn(*d, generator=g, device="cuda").to(torch.bfloat16)
    idx = torch.rand(U, 128, generator=g, device="cuda").argsort(-1)[:, :T].sort(-1).values.to(torch.int16).contiguous()
    q, k1, x = rnd(U, G, 128), torch.zeros(U, 128, device="cuda", dtype=torch.bfloat16), rnd(U, 128)
    k1.scatter_(1, idx.long(), rnd(U, T))
    c0 = idx[:, :1].long()
    k1.scatter_(1, c0, torch.ones_like(c0, dtype=torch.bfloat16))        # one kept channel: 1 in the first row,
    k2 = k1.clone()
    k2.scatter_(1, c0, torch.full_like(c0, 1 + 2**-7, dtype=torch.bfloat16))   # the next bf16 in the second
    keys, vals = torch.stack([k1, k2], 1), torch.stack([x, -x], 1)       # [U, 2, 128]
    S = 1 if second_row == "tail" else 2
    kp = torch.full((U, S, pitch), float("nan"), device="cuda", dtype=torch.bfloat16)
    kp[..., :T] = keys[:, :S].gather(2, idx.long()[:, None].expand(U, S, T))
    kt, vt = keys[:, 1:].contiguous(), vals[:, 1:].contiguous()
    shape = thk.make_shape(1, U, G, 1, 128, S, 1, T, ld, thk.THK_BF16, 1)
    assert thk.thk_decode_on_matrix_cores(shape) == 1
    out = torch.full_like(q, float("nan"))
    ws = ws_tensor(thk.thk_workspace_bytes(shape, thk.THK_OP_DECODE))
    tail = (kt, vt, 1, 1) if second_row == "tail" else (None, None, 0, 0)
    if second_row == "pruned values":
        iv = torch.arange(128, device="cuda", dtype=torch.int16).repeat(U, 1)
        thk.thk_decode_attn_kv(shape, q, kp, idx, vals, iv, 128, 128, None, None, 0, 0, out, ws)
    else:
        thk.thk_decode_attn(shape, q, kp, idx, vals[:, :S].contiguous(), *tail, out, ws)
    qk = torch.zeros(U, G, 128, dtype=torch.float64, device="cuda")
    il = idx.long()[:, None].expand(U, G, T)
    qk.scatter_(2, il, q.double().gather(2, il))
    qs = torch.stack([qk, q.double() if second_row == "tail" else qk], 2)          # the query each row meets
    p = torch.softmax((qs * keys.double()[:, None]).sum(-1) / 128 ** 0.5, -1)      # [U, G, 2]
    ref = (p[..., None] * vals.double()[:, None]).sum(2)
    size = (p[..., None] * vals.double().abs()[:, None]).sum(2)
    worst = ((out.double() - ref).abs() / (2**-8 * ref.abs() + 2**-20 * size)).max().item()
    print(f"error over its bound: {worst:.3f}")
    assert worst <= 1



@pytest.mark.parametrize("levels", [1, 2])
def test_prune_single_launch_with_late_query_norms(levels, thk_env):
    """The prologue publishes the query norms after the arrival counters, so a unit's sums can be complete before
    its norms are there: held back from the host here, once behind blocks that wait for the list and once behind
    blocks that give up at once.  A block that finds no norms in all its looks (THK_PRUNE_NORM_POLLS=1) must
    not score with zeros: the scores are NaN, the list is one of valid channels, and the next call is right."""
    thk_env.setenv("THK_PRUNE_LAUNCH", "solo")
    if levels == 2:                                # 102 blocks of 128 rows per unit
        thk_env.setenv("THK_PRUNE_BLOCK_ROWS", "128")
    L, B, N, G, S, S_obs, T = (2, 2, 4, 2, 3000, 32, 76) if levels == 1 else (1, 2, 2, 1, 13008, 32, 64)
    U = L * B * N
    shape = thk.make_shape(L, B, N * G, N, D, S, S_obs, T, 0, thk.THK_BF16, 0)
    assert thk.thk_prune_launches(shape) == 1
    for rep, (delay, spin, polls) in enumerate([(200, None, None), (200, "0", None), (500, None, "1"), (0, None, None)]):
        thk_env.setenv("THK_PRUNE_NORM_DELAY_US", str(delay))
        for name, value in (("THK_PRUNE_SPIN_LIMIT", spin), ("THK_PRUNE_NORM_POLLS", polls)):
            if value is None:
                thk_env.delenv(name, raising=False)
            else:
                thk_env.setenv(name, value)
        q_obs = _randn((L, B, N * G, S_obs, D), "bf16", 271 + rep, 1.0)
        k = _randn((L, B, N, S, D), "bf16", 281 + rep, 1.0)
        score, idx, kp = gpu_prune(shape, q_obs, k)
        if polls is not None:
            assert score.isnan().all() and (idx >= 0).all() and (idx < D).all()
            continue
        o_sc, o_idx, _ = oracle_prune(q_obs, k, "bf16", T)
        rel = np.abs(score.cpu().numpy().astype(np.float64) - o_sc.reshape(U, D)) / o_sc.reshape(U, D)
        assert rel.max() <= SCORE_TOL
        check_idx_with_tie_rule(idx.cpu().numpy(), o_idx, o_sc, T)
        np.testing.assert_array_equal(as_numpy(kp), O.compact_keys(as_numpy(k).reshape(U, S, D), idx.cpu().numpy(), "bf16"))



def test_prune_blocks_of_short_calls_wait_as_long_as_those_of_long_calls(thk_env):
    """A block resigns after THK_PRUNE_SPIN_LIMIT polls of about half a microsecond, in calls of one round too, where it
    looks twice as often: 1800 of them outlast norms that come 500 us late.  The give-up counters lie behind the
    partial sums, the norms and two other counters, 256 bytes a unit; the finisher's closing ticket is 2^24."""
    thk_env.setenv("THK_PRUNE_LAUNCH", "solo")
    thk_env.setenv("THK_PRUNE_BLOCK_ROWS", "128")
    thk_env.setenv("THK_PRUNE_NORM_DELAY_US", "500")
    U, S, NB = 2, 3000, 24
    shape = thk.make_shape(1, 1, U, U, D, S, 32, 64, 0, thk.THK_BF16, 0)
    q_obs, k = _randn((1, 1, U, 32, D), "bf16", 291, 1.0), _randn((1, 1, U, S, D), "bf16", 292, 1.0)
    score = torch.empty(U, D, dtype=torch.float32, device="cuda")
    idx = torch.empty(U, 64, dtype=torch.int16, device="cuda")
    kp = torch.empty(U, S, 64, dtype=torch.bfloat16, device="cuda")
    first = U * NB * D * 8 + U * D * 8 + 2 * U * 256
    resigned = {}
    for spin in ("1800", "0"):
        thk_env.setenv("THK_PRUNE_SPIN_LIMIT", spin)
        ws = ws_tensor(thk.thk_workspace_bytes(shape, thk.THK_OP_PRUNE))
        thk.thk_prune(shape, q_obs, k, score, idx, kp, ws)
        torch.cuda.synchronize()
        resigned[spin] = (ws[first:first + U * 256].view(torch.int32)[::64] - (1 << 24)).tolist()
    assert resigned == {"1800": [0] * U, "0": [NB - 1] * U}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("S", [100, 700, 9000])
def test_prune_query_norms_keep_53_bits(S, dtype, prune_launch):
    """Three heads whose norms are 1, 2^-24 and 2^-52: their sum needs the last bit of an fp64, and with it the
    score lies just above the middle of two fp32 numbers (without it, on the middle, which rounds down)."""
    U, G = 2, 3
    q_obs = torch.tensor([1.0, 2.0**-24, 2.0**-52], device="cuda").repeat(U)[None, None, :, None, None].expand(1, 1, U * G, 1, D)
    k = torch.zeros(1, 1, U, S, D, device="cuda")
    k[:, :, :, S // 2] = 1.0
    shape = thk.make_shape(1, 1, U * G, U, D, S, 1, 64, 0, DT[dtype], 0)
    score, idx, _ = gpu_prune(shape, q_obs.to(TDT[dtype]).contiguous(), k.to(TDT[dtype]))
    assert (score == 1 + 2.0**-23).all()
    assert (idx.cpu() == torch.arange(64, dtype=torch.int16)).all()      # all tie: the lowest channels


@pytest.mark.parametrize("U,G", [(8388601, 9), (8388607, 16)])
def test_decode_grid_rounded_to_eights_stays_within_one_launch(U, G):
    """Units whose head groups come to just under 2^24 blocks, the most that one launch may have: laid out in eights they
    must not be more.  One row each, so every head's output is that row."""
    q = torch.zeros(U, G, 128, device="cuda", dtype=torch.bfloat16)
    kp = torch.ones(U, 1, 4, device="cuda", dtype=torch.bfloat16)
    v = (torch.arange(U, device="cuda") % 251).to(torch.bfloat16)[:, None, None].expand(U, 1, 128).contiguous()
    idx = torch.arange(4, device="cuda", dtype=torch.int16).repeat(U, 1)
    out = torch.full_like(q, -1.0)
    shape = thk.make_shape(1, 1, U * G, U, 128, 1, 1, 4, 0, thk.THK_BF16, 1)
    thk.thk_decode_attn(shape, q, kp, idx, v, None, None, 0, 0, out, ws_tensor(16))
    torch.cuda.synchronize()
    assert (out[:, 0] == v[:, 0]).all() and (out[:, G - 1] == v[:, 0]).all()
    assert (out[:, 1:, 0] == v[:, 0, :1]).all()


def test_launch_of_more_work_items_than_the_runtime_counts_is_refused():
    """2^24 + 8 units of one row would be launched as 8 blocks."""
    U = (1 << 24) + 8
    q = torch.zeros(U, 1, 128, device="cuda", dtype=torch.bfloat16)
    kp = torch.ones(U, 1, 4, device="cuda", dtype=torch.bfloat16)
    idx = torch.arange(4, device="cuda", dtype=torch.int16).repeat(U, 1)
    shape = thk.make_shape(1, 1, U, U, 128, 1, 1, 4, 0, thk.THK_BF16, 1)
    with pytest.raises(thk.ThkError, match="status 6"):
        thk.thk_decode_attn(shape, q, kp, idx, torch.ones_like(q), None, None, 0, 0, torch.empty_like(q), ws_tensor(16))
