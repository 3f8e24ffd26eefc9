"""The routes a call takes through the alignment kernel, each at the sizes where
it begins and ends, bit for bit against the oracle: workgroups of 126 rows
(one, two, more than the boundary regions hold apart), walks from whole step
masks, whole descent bytes, blocks, banded windows and windows of whole chunks, the path written by the
sweep workgroups (small batches) and by path writers (large ones), with rows
and pointers that are not 16-byte aligned."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

CASES = [
    # B, T, S, lengths: what it reaches
    (3, 1, 37, [(1, 37), (1, 1), (0, 5)]),                       # one row; an empty item
    (2, 126, 126, [(126, 126), (125, 126)]),                     # one full workgroup, forced diagonal
    (3, 127, 211, [(127, 211), (126, 127), (64, 64)]),           # a second workgroup of one row
    (2, 253, 1001, [(253, 1001), (252, 999)]),                   # three workgroups, whole step masks
    (2, 300, 2503, [(300, 2503), (190, 2500)]),                  # whole descent bytes
    (2, 505, 1999, [(505, 1999), (504, 1500)]),                  # workgroups that share a boundary region
    (2, 1010, 4101, [(1010, 4101), (700, 3333)]),                # blocks of descent bytes
    (1, 2400, 6000, [(2400, 6000)]),                             # ... three blocks of four chunks in LDS
    (2, 3024, 3500, [(3024, 3500), (2900, 3400)]),               # ... the tallest item three blocks hold
    (1, 3025, 3500, [(3025, 3499)]),                             # banded windows from one row more on
    (1, 4300, 4400, [(4300, 4390)]),                             # banded windows
    (1, 2, 530_000, [(2, 530_000)]),                             # few rows, a record past LDS: windows of whole chunks
    (1, 2, 1_100_000, [(2, 1_100_000)]),                         # ... with more than 2^15 chunks
    (16, 1010, 4160, None),                                      # more cells than the sweep workgroups write
]


@pytest.mark.parametrize("B,T,S,lengths", CASES)
@pytest.mark.parametrize("shift", [0, 1])
def test_routes(B, T, S, lengths, shift):
    import paper_2409_07704_amd as mas

    if lengths is None:
        if shift:
            pytest.skip("one alignment is enough for the large batch")
        lengths = [(T - 61 * b, S - 37 * b) for b in range(B)]
    tx, ty = (np.array(v, dtype=np.int32) for v in zip(*lengths))
    value, tx, ty = synth.normal_batch(B, T, S, tx, ty, seed=B * T + S)
    print(f"[gpu-case] routes B={B} T={T} S={S} shift={shift}", flush=True)
    op, os_, ost = oracle.mas(value, tx, ty)
    n = value.size
    # value `shift` floats and the path `shift` bytes off their allocations
    v = torch.empty(n + 4, dtype=torch.float32, device="cuda")[shift : shift + n].view(B, T, S)
    v.copy_(torch.from_numpy(value))
    raw = torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    path = raw[16 + shift : 16 + shift + n].view(B, T, S)
    x, y = torch.from_numpy(tx).cuda(), torch.from_numpy(ty).cuda()
    score = torch.full((B,), 3.0, device="cuda")
    status = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    rs = torch.full((B, T + 1), -7, dtype=torch.int32, device="cuda")
    dur = torch.full((B, T), -7, dtype=torch.int32, device="cuda")
    ws = mas.Workspace(B, T, S)
    for _ in range(2):
        mas.mas_forward_ex(v, x, y, path, score, status, workspace=ws)
        mas.mas_search(v, x, y, rs, workspace=ws, durations_out=dur)
    torch.cuda.synchronize()
    assert np.array_equal(status.cpu().numpy(), ost)
    assert score.cpu().numpy().tobytes() == os_.tobytes()
    assert np.array_equal(path.cpu().numpy(), op)
    edge = raw.cpu().numpy()
    assert (edge[: 16 + shift] == 0xA5).all() and (edge[16 + shift + n :] == 0xA5).all()
    assert np.array_equal(dur.cpu().numpy(), op.sum(axis=2, dtype=np.int32))
    assert np.array_equal(rs.cpu().numpy()[:, 1:] - rs.cpu().numpy()[:, :-1], dur.cpu().numpy())


@pytest.mark.parametrize("B,T,S", [(2, 505, 1999), (17, 1010, 4160)])
def test_generation_starts_over(B, T, S):
    """The last generations of a workspace and the first ones after them: no tag
    of a call is 0, the value of the boundary words of a clear workspace (items
    of five and nine workgroups, which use both tags of a call; a small batch
    and one with narrow polls)."""
    import paper_2409_07704_amd as mas

    tx = np.array([T - 5 * (b % 16) for b in range(B)], np.int32)
    ty = np.array([S - 37 * b for b in range(B)], np.int32)
    value, tx, ty = synth.normal_batch(B, T, S, tx, ty, seed=S)
    print(f"[gpu-case] generation starts over B={B} T={T} S={S}", flush=True)
    op, os_, ost = oracle.mas(value, tx, ty)
    v, x, y = (torch.from_numpy(a).cuda() for a in (value, tx, ty))
    ws = mas.Workspace(B, T, S)
    off = ws.ptr - ws._buf.data_ptr()
    gen = ws._buf[off : off + 4].view(torch.int32)
    assert gen.item() == 0
    gen.fill_(0x7FFFFFFD)
    seen = []
    for _ in range(4):
        path = torch.full((B, T, S), 0xA5, dtype=torch.uint8, device="cuda")
        score = torch.full((B,), 3.0, device="cuda")
        status = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        mas.mas_forward_ex(v, x, y, path, score, status, workspace=ws)
        torch.cuda.synchronize()
        seen.append(gen.item())
        assert np.array_equal(status.cpu().numpy(), ost)
        assert score.cpu().numpy().tobytes() == os_.tobytes()
        assert np.array_equal(path.cpu().numpy(), op)
    assert seen == [0x7FFFFFFE, 0, 1, 2]


@pytest.mark.parametrize("B,T,S,shift", [
    (16, 1010, 4160, 1),    # whole pieces, all of them off a boundary
    (16, 1010, 4171, 0),    # every row at another place between boundaries
    (16, 1010, 4171, 3),
    (70_000, 31, 33, 0),    # two or one pieces a row
    (440_000, 12, 13, 5),   # rows of less than a piece
])
def test_path_writers_unaligned(B, T, S, shift):
    """The path writers' pieces and single bytes, in batches of more cells than
    the sweep workgroups write: every byte against the oracle, with bytes on
    both sides of the path left alone."""
    import paper_2409_07704_amd as mas

    rng = np.random.default_rng(B + S + shift)
    tx = rng.integers(1, T + 1, B).astype(np.int32)
    ty = rng.integers(tx, S + 1).astype(np.int32)
    tx[0], ty[0], tx[1] = T, S, 0
    value, tx, ty = synth.normal_batch(B, T, S, tx, ty, seed=S)
    print(f"[gpu-case] path writers B={B} T={T} S={S} shift={shift}", flush=True)
    op, os_, ost = oracle.mas(value, tx, ty)
    n = value.size
    assert n > 64 << 20
    v, x, y = (torch.from_numpy(a).cuda() for a in (value, tx, ty))
    raw = torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    path = raw[16 + shift : 16 + shift + n].view(B, T, S)
    status = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    mas.mas_forward_ex(v, x, y, path, None, status, workspace=mas.Workspace(B, T, S))
    torch.cuda.synchronize()
    assert np.array_equal(status.cpu().numpy(), ost)
    assert np.array_equal(path.cpu().numpy(), op)
    edge = raw.cpu().numpy()
    assert (edge[: 16 + shift] == 0xA5).all() and (edge[16 + shift + n :] == 0xA5).all()


def test_more_workgroups_than_a_grid_holds():
    """4.3 M items of 127 padded rows: two workgroups each, more threads than one
    launch can have.  One-token items have closed-form results."""
    import paper_2409_07704_amd as mas

    B, T, S = 4_300_000, 127, 1
    print(f"[gpu-case] large grid B={B} T={T} S={S}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    value = torch.randn((B, T, S), generator=gen, device="cuda")
    x = torch.ones(B, dtype=torch.int32, device="cuda")
    y = torch.ones_like(x)
    x[::1000] = 2  # infeasible
    y[1::1000] = 0  # empty
    ok = (x == 1) & (y == 1)
    want = torch.where(y == 0, 1, torch.where(x == 2, 2, 0)).to(torch.int32)
    score = torch.full((B,), 3.0, device="cuda")
    status = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    ws = mas.Workspace(B, T, S)
    for _ in range(2):
        rs = torch.full((B, T + 1), -7, dtype=torch.int32, device="cuda")
        mas.mas_search(value, x, y, rs, score, status, workspace=ws)
        assert torch.equal(status, want)
        assert torch.equal(score, torch.where(ok, value[:, 0, 0], -torch.inf))
        assert (rs[:, 0] == 0).all() and (rs[:, 1:] == ok[:, None].to(torch.int32)).all()
    del rs
    path = torch.full((B, T, S), 0xA5, dtype=torch.uint8, device="cuda")
    status.fill_(-1)
    mas.mas_forward_ex(value, x, y, path, score, status, workspace=ws)
    assert torch.equal(status, want)
    assert torch.equal(path[:, 0, 0].bool(), ok) and not path[:, 1:].any()
