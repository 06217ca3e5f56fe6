"""The tiles a wavefront of the decode kernels takes: 32-row tiles of its piece, then 16-row tiles of the tail,
each asked for through a range that ends with the tile.  Sequence lengths and tail lengths around the tiles'
edges, pieces without rows and waves without tiles, with NaN in every row behind the sequence and
behind the tail: what a tile reads past its last row must not count."""
import numpy as np
import pytest
import torch

import paper_2407_21018_amd as thk
from oracle import oracle as O
from paper_2407_21018_amd.synth import as_numpy
from helpers import ATTN_TOL, DT, TDT, attn_rel_err, ws_tensor

pytestmark = pytest.mark.gpu
D, CAP = 128, 112


def _kept(rng, U, T):
    return np.stack([np.sort(rng.permutation(D)[:T]) for _ in range(U)]).astype(np.int16)


@pytest.mark.parametrize("tail", [0, 1, 16, 17, 112])
@pytest.mark.parametrize("dtype,G,T,T_v", [("bf16", 1, 76, 0), ("bf16", 2, 51, 0), ("bf16", 1, 64, 68), ("bf16", 4, 64, 0), ("bf16", 3, 51, 0),
                                           ("bf16", 8, 100, 0), ("bf16", 8, 76, 44), ("f32", 1, 64, 0), ("f32", 4, 51, 0), ("f32", 2, 76, 128)])
def test_decode_tile_edges(dtype, G, T, T_v, tail, decode_merge):
    B, N_kv = 1, 3
    U, N_q = B * N_kv, N_kv * G
    rng = np.random.default_rng(1000 * tail + 10 * T + G)
    idx_np, idxv_np = _kept(rng, U, T), _kept(rng, U, max(T_v, 1))
    for S, n_split in [(1, 1), (31, 2), (32, 1), (33, 1), (127, 1), (129, 3), (160, 2), (449, 4), (1000, 16)]:
        S_cap = S + 40
        g = torch.Generator(device="cuda"); g.manual_seed(S)
        rnd = lambda *shape: torch.randn(*shape, generator=g, device="cuda").to(TDT[dtype])
        q, kp, v = rnd(B, N_q, D), rnd(U, S_cap, T), rnd(U, S_cap, T_v or D)
        kt, vt = rnd(U, CAP, D), rnd(U, CAP, D)
        for x, n in ((kp, S), (v, S), (kt, tail), (vt, tail)):
            x[:, n:] = float("nan")
        idx, idxv = torch.from_numpy(idx_np).cuda(), torch.from_numpy(idxv_np).cuda()
        shape = thk.make_shape(1, B, N_q, N_kv, D, S, 1, T, 0, DT[dtype], n_split, 0, S_cap)
        out = torch.empty(B * N_q, D, dtype=q.dtype, device="cuda")
        ws = ws_tensor(thk.thk_workspace_bytes(shape, thk.THK_OP_DECODE))
        if T_v:
            thk.thk_decode_attn_kv(shape, q, kp, idx, v, idxv, T_v, T_v, kt, vt, tail, CAP, out, ws)
        else:
            thk.thk_decode_attn(shape, q, kp, idx, v, kt, vt, tail, CAP, out, ws)
        torch.cuda.synchronize()
        h = lambda x, n: as_numpy(x[:, :n].contiguous()).reshape(B, N_kv, n, x.shape[-1])
        tails = (h(kt, tail), h(vt, tail), tail) if tail else ()
        if T_v:
            ref = O.decode_attn_kv(as_numpy(q), h(kp, S), idx_np.reshape(B, N_kv, T), h(v, S), idxv_np.reshape(B, N_kv, T_v), dtype, *tails)
        else:
            ref = O.decode_attn(as_numpy(q), h(kp, S), idx_np.reshape(B, N_kv, T), h(v, S), dtype, *tails)
        err = attn_rel_err(out, ref.reshape(-1, D)).max()
        assert err <= ATTN_TOL[dtype], f"S={S} n_split={n_split}: {err}"


# the merge launch: a wave takes 16 pieces at a time, one, four or eight waves a head; 130 pieces are a second turn of
# the first wave's, and 70 pieces of 64 rows leave most of 130 without rows
@pytest.mark.parametrize("n_split", [2, 15, 16, 17, 33, 63, 64, 65, 128, 130, 300])
@pytest.mark.parametrize("dtype,G,T", [("bf16", 4, 64), ("f32", 1, 51)])
def test_decode_merge_launch_piece_counts(dtype, G, T, n_split, thk_env):
    thk_env.setenv("THK_DECODE_MERGE", "kernel")
    B, N_kv = 1, 2
    for S in (64 * min(n_split, 140), 4450):
        g = torch.Generator(device="cuda"); g.manual_seed(S + n_split)
        rnd = lambda *shape: torch.randn(*shape, generator=g, device="cuda").to(TDT[dtype])
        idx_np = _kept(np.random.default_rng(n_split), N_kv, T)
        q, kp, v = 4 * rnd(B, N_kv * G, D), rnd(N_kv, S, T), rnd(N_kv, S, D)
        shape = thk.make_shape(1, B, N_kv * G, N_kv, D, S, 1, T, 0, DT[dtype], n_split)
        out = torch.empty(N_kv * G, D, dtype=q.dtype, device="cuda")
        ws = ws_tensor(thk.thk_workspace_bytes(shape, thk.THK_OP_DECODE))
        ws.fill_(255)   # NaN where a piece leaves no record, and behind the last one
        thk.thk_decode_attn(shape, q, kp, torch.from_numpy(idx_np).cuda(), v, None, None, 0, 0, out, ws)
        torch.cuda.synchronize()
        h = lambda y: as_numpy(y).reshape(B, N_kv, S, y.shape[-1])
        ref = O.decode_attn(as_numpy(q), h(kp), idx_np.reshape(B, N_kv, T), h(v), dtype)
        err = attn_rel_err(out, ref.reshape(-1, D)).max()
        assert err <= ATTN_TOL[dtype], f"S={S} n_split={n_split}: {err}"


# calls of a block per 64 rows: the shortest, a last piece of one row, the most blocks (256; of eight heads and of fp32 in narrow rows 448,
# which only calls with a tail take), and one row more, where pieces have whole steps again; with a workspace that holds half of the
# pieces the call takes those
@pytest.mark.parametrize("dtype,N_q,N_kv,S,pieces", [("bf16", 32, 8, 513, 9), ("bf16", 32, 8, 2048, 32), ("bf16", 32, 8, 2049, None), ("bf16", 8, 4, 961, 16),
                                                     ("bf16", 16, 2, 4033, 64), ("f32", 8, 8, 705, 12), ("f32", 8, 8, 2048, 32), ("f32", 8, 2, 1025, 17),
                                                     ("bf16", 56, 8, 3553, 56), ("bf16", 56, 8, 3585, None), ("f32", 9, 9, 129, 3), ("f32", 8, 8, 2779, 44), ("f32", 8, 8, 3585, None)])
@pytest.mark.parametrize("tail", [0, 1, 112])
def test_decode_pieces_of_half_steps(dtype, N_q, N_kv, S, pieces, tail):
    T, G = 76, N_q // N_kv
    shape = thk.make_shape(1, 1, N_q, N_kv, D, S, 1, T, 0, DT[dtype], 0)
    n = thk.thk_default_split(shape, thk.THK_OP_DECODE)
    assert n == pieces if pieces else n < -(-S // 64)
    g = torch.Generator(device="cuda"); g.manual_seed(S)
    rnd = lambda *shape: torch.randn(*shape, generator=g, device="cuda").to(TDT[dtype])
    idx_np = _kept(np.random.default_rng(S), N_kv, T)
    q, kp, v, kt, vt = 3 * rnd(N_q, D), rnd(N_kv, S, T), rnd(N_kv, S, D), rnd(N_kv, CAP, D), rnd(N_kv, CAP, D)
    h = lambda y, m: as_numpy(y[:, :m].contiguous()).reshape(1, N_kv, m, y.shape[-1])
    tails = (h(kt, tail), h(vt, tail), tail) if tail else ()
    ref = O.decode_attn(as_numpy(q).reshape(1, N_q, D), h(kp, S), idx_np.reshape(1, N_kv, T), h(v, S), dtype, *tails).reshape(-1, D)
    need = thk.thk_workspace_bytes(shape, thk.THK_OP_DECODE)
    for held in (need, need // 2):
        out = torch.empty(N_q, D, dtype=q.dtype, device="cuda")
        ws = ws_tensor(held)[:held]
        ws.fill_(255)
        thk.thk_decode_attn(shape, q, kp, torch.from_numpy(idx_np).cuda(), v, kt, vt, tail, CAP, out, ws)
        torch.cuda.synchronize()
        err = attn_rel_err(out, ref).max()
        assert err <= ATTN_TOL[dtype], f"workspace of {held}: {err}"
