"""The mask kernels on both sides of the lines that choose how a row is split."""
import numpy as np
import pytest
import torch

from paper_2509_16518_amd import fgattn as F
from gpu_util import say

pytestmark = pytest.mark.gpu


def problem(H, L, d, M, N, seed, flags=0, scale=1.0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    q, k = (torch.randn((1, H, L, d), generator=gen, device="cuda").bfloat16() for _ in range(2))
    p = F.make_params(q, k, k, q, M, N, scale * d ** -0.5, flags)
    ws = torch.empty(F.fgattn_mask_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    return q, k, p, ws, torch.empty(H * ((L + M - 1) // M) + 1, dtype=torch.int64, device="cuda")


def emitted(p, ws, indptr):
    ids = torch.zeros(max(int(indptr[-1]), 1), dtype=torch.int32, device="cuda")
    F.fgattn_mask_emit(p, indptr, ids, ws)
    return ids[:int(indptr[-1])]


def kept_rows(p, ws, indptr, G):
    """The kept set as [rows, G] truth values, from the emitted ids."""
    rows = indptr.numel() - 1
    row = torch.repeat_interleave(torch.arange(rows, device="cuda"), indptr[1:] - indptr[:-1])
    kept = torch.zeros((rows, G), dtype=torch.bool, device="cuda")
    kept[row, emitted(p, ws, indptr).long()] = True
    return kept


# one wave per row and several (few long rows), rows that end inside a pair of words, inside a batch of 32 words and at its
# edges, outputs that start at every place of a 16-byte group, and buffers that end early
@pytest.mark.parametrize("H,L,M,N", [(1, 40000, 128, 1), (1, 8192, 128, 1), (2, 4128, 16, 1), (1, 1024, 16, 1), (1, 1056, 16, 1),
                                     (3, 2080, 64, 1), (1, 100, 16, 1), (2, 31, 16, 1), (1, 4000, 16, 1), (1, 1100, 64, 1)])
def test_emitted_ids_are_the_bits_in_order(H, L, M, N):
    # Which ids a row keeps is known beforehand: query block r looks at column r % 64, where a key holds +1 or -1.  Scores are 64 or
    # -64, so the +1 keys share the whole mass equally and top_p = 1 keeps every one of them and nothing else.
    q, k, _, ws, indptr = problem(H, L, 64, M, N, seed=L)
    QB = (L + M - 1) // M
    q.zero_()
    q[:, :, torch.arange(L), torch.arange(L) // M % 64] = 64.0
    k.copy_(torch.where(k > -0.5, 1.0, -1.0))
    p = F.make_params(q, k, k, q, M, N, 1.0)
    F.fgattn_mask_select(q, k, p, 1.0, indptr, ws)
    bits = (k[0][:, :, torch.arange(QB) % 64] > 0).transpose(1, 2).reshape(H * QB, L)
    want = bits.nonzero()[:, 1].int()
    rows, G = H * QB, L
    assert torch.equal(indptr[1:] - indptr[:-1], bits.sum(1))
    assert torch.equal(indptr[1:], bits.sum(1).cumsum(0)) and int(indptr[0]) == 0
    nnz = want.numel()
    say("    %d rows of %d, %d ids" % (rows, G, nnz))
    for offset in range(4):
        for cap in (nnz, nnz - 1, nnz - 3, nnz // 2 + 1):
            cap = max(cap, 0)
            buf = torch.full((nnz + 16,), -7, dtype=torch.int32, device="cuda")
            F.fgattn_mask_emit(p, indptr, buf[offset:offset + cap], ws)
            assert torch.equal(buf[offset:offset + cap], want[:cap]), (offset, cap)
            assert (buf[:offset] == -7).all() and (buf[offset + cap:] == -7).all(), (offset, cap)


# outputs that start at every place of a 128-byte line and end early; rows that keep everything (eight ids in every byte), long
# runs of nothing between single ids, and every byte there is
@pytest.mark.parametrize("L,M", [(3000, 128), (1024, 16), (1025, 16), (33, 16)])
def test_emitted_ids_at_every_place_of_a_line(L, M):
    q, k, p, ws, indptr = problem(1, L, 64, M, 1, seed=L)
    j = torch.arange(L, device="cuda")
    for on in (torch.ones_like(j, dtype=torch.bool), (j % 700 == 5) | (j == L - 1), (((j // 8) >> (j % 8)) & 1 != 0) | (j == 0)):
        # query blocks hold e_0 and keys +1 or -1 in column 0: scores 64 and -64, so top_p = 1 keeps exactly the former
        q.zero_()
        q[..., 0] = 64.0
        k.copy_(torch.where(on, 1.0, -1.0)[None, None, :, None].expand_as(k))
        p = F.make_params(q, k, k, q, M, 1, 1.0)
        F.fgattn_mask_select(q, k, p, 1.0, indptr, ws)
        want = on.nonzero()[:, 0].int().repeat((L + M - 1) // M)
        nnz = want.numel()
        assert int(indptr[-1]) == nnz
        for offset in range(32):
            cap = nnz - offset % 3
            buf = torch.full((nnz + 64,), -7, dtype=torch.int32, device="cuda")
            F.fgattn_mask_emit(p, indptr, buf[offset:offset + cap], ws)
            assert torch.equal(buf[offset:offset + cap], want[:cap]), offset
            assert (buf[:offset] == -7).all() and (buf[offset + cap:] == -7).all(), offset


# fewer than eight stretches of key blocks, eight, and counts off a multiple of eight; one score tile, more than share a
# stretch, tiles whose last rows or whole waves are past the end, chunks that begin inside a slice; key blocks past the end
# of a tile of 32; means that are all negative or far apart, so that a padded position would show in a row's range
@pytest.mark.parametrize("H,L,d,M,N,one_tile", [(1, 3500, 64, 16, 1, False), (3, 4099, 128, 128, 1, False), (2, 4609, 64, 16, 1, True),
                                                (11, 4100, 128, 32, 1, False), (1, 20000, 64, 16, 1, False), (5, 2050, 128, 64, 8, False)])
def test_scores_of_every_tile_and_stretch(H, L, d, M, N, one_tile):
    q, k, p, ws, indptr = problem(H, L, d, M, N, seed=L + 1, flags=F.FLAG_MASK_ONE_TILE_CHUNKS if one_tile else 0, scale=3.0)
    q -= 2.0   # (means of one sign)
    k += 2.0
    F.fgattn_mask_select(q, k, p, 0.9, indptr, ws)
    rows, G = indptr.numel() - 1, (L + N - 1) // N
    QB = rows // H
    got = kept_rows(p, ws, indptr, G).view(H, QB, G)

    def means(x, n):
        pad = torch.nn.functional.pad(x.double(), (0, 0, 0, (-L) % n)).view(H, -1, n, d).sum(2)
        count = torch.full((pad.shape[1], 1), float(n), device="cuda", dtype=torch.float64)
        count[-1] = L - (pad.shape[1] - 1) * n
        return (pad / count).float().bfloat16().double()
    s = (means(q[0], M) @ means(k[0], N).transpose(1, 2)) * p.scale
    prob = torch.softmax(s, -1)
    mass = (prob * got).sum(-1)
    # the kept set reaches p, and not without its least probable member; and it is a top set: no key block left out is more
    # probable than one kept (both up to the rounding of fp32 scores and of the means to bf16, whose fp32 sums may differ in the
    # last bit from the exact ones here)
    tol = 1e-5 if M * N == 16 else 2e-2
    least = torch.where(got, prob, 2.0).amin(-1)
    most_out = torch.where(got, -1.0, prob).amax(-1)
    assert (mass >= 0.9 - tol).all() and (mass - least < 0.9 + tol).all(), (mass.min(), (mass - least).max())
    assert (most_out <= least * (1 + (1e-4 if tol < 1e-4 else 0.3)) + 1e-9).all(), float((most_out / least).max())


# The selection that a row of this length takes (by a wave, from bytes, or without kept scores), against the one that reads it in
# every pass.  Rows of scores that are spread out, that leave most weights zero, that take a few values only, that sit close
# together beside one dominant score, and that are all equal: from few members of the crossing bin to more than any kernel
# keeps.  Rows end at, before and after a group of sixteen, a word, and the largest row of a kernel.
@pytest.mark.parametrize("G", [1, 15, 147, 257, 1000, 4096, 4097, 8195, 32768, 32769, 65536, 65537, 118800, 131072, 131073])
def test_selection_from_bytes_equals_selection_from_memory(G):
    compare_with_selection_from_memory(G, 0)


# Score tiles one by one leave every length to the kernels that read a row once, up to their longest, and to the general one above
@pytest.mark.parametrize("G", [1, 15, 147, 257, 1000, 1025, 4096, 4097, 32768, 32769, 65536, 65537, 118800, 131071, 131072, 131073])
def test_selection_from_bytes_of_single_tiles_equals_selection_from_memory(G):
    compare_with_selection_from_memory(G, F.FLAG_MASK_ONE_TILE_CHUNKS)


def compare_with_selection_from_memory(G, flags_of_first):
    d, M = 64, 128
    for kind in ("spread", "peaked", "few values", "close", "equal"):
        for top_p in (0.3, 0.9, 1.0):
            res = []
            for flags in (flags_of_first, F.FLAG_MASK_ROWS_IN_HBM):
                q, k, _, ws, indptr = problem(1, G, d, M, 1, seed=G, flags=flags)
                if kind == "few values":
                    k = (k[..., :1] > 0.5).to(k.dtype).expand_as(k).contiguous()
                elif kind == "close":
                    k = 1.0 + (k > 1.0).to(k.dtype) * 2.0 ** -7
                    k[:, :, G // 2] = 40.0
                    q = q.abs()
                elif kind == "equal":
                    k = torch.ones_like(k)
                p = F.make_params(q, k, k, q, M, 1, (20.0 if kind == "peaked" else 1.0) * d ** -0.5, flags)
                F.fgattn_mask_select(q, k, p, top_p, indptr, ws)
                res.append((indptr, emitted(p, ws, indptr)))
            assert torch.equal(res[0][0], res[1][0]), (kind, top_p)
            assert torch.equal(res[0][1], res[1][1]), (kind, top_p)


# Rows with more members than a workgroup keeps come after its other rows: several rows per workgroup of each kernel size, of
# which none, some or all are such rows (heads of equal keys between heads of ordinary ones)
@pytest.mark.parametrize("H,L,M", [(20, 2000, 16), (3, 8195, 16), (2, 40000, 64), (2, 70000, 128)])
def test_overfull_rows_among_others(H, L, M):
    overfull_rows_among_others(H, L, 64, M)


# rows beyond 65536 that are few enough for kept scores, several to a workgroup
def test_overfull_rows_among_others_in_the_longest_rows():
    overfull_rows_among_others(2, 66000, 128, 128)


def overfull_rows_among_others(H, L, d, M):
    for full in ([], list(range(0, H, 2)), list(range(H))):
        res = []
        for flags in (0, F.FLAG_MASK_ROWS_IN_HBM):
            q, k, p, ws, indptr = problem(H, L, d, M, 1, seed=L + len(full), flags=flags)
            k[:, full] = 1.0
            F.fgattn_mask_select(q, k, p, 0.9, indptr, ws)
            res.append((indptr, emitted(p, ws, indptr)))
        assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1]), full


# Many long rows go without a buffer of scores: against the kernel that reads kept scores in every pass.  Rows and key blocks
# off every multiple of a tile, a wave and a workgroup; the shortest rows that go this way and rows longer than any kernel keeps in LDS;
# key block means and K in place, in either storage order; one chunk of slices and two; scores that are spread out, mostly
# without weight, of negative scale, and, in every other head, crowded beside a few large ones (lists that overflow).
@pytest.mark.parametrize("B,H,L,d,M,N,tokens_first", [(1, 1, 33000, 64, 16, 1, False), (2, 3, 15001, 128, 16, 1, True), (1, 7, 40000, 128, 128, 1, True),
                                                      (1, 2, 131073, 64, 128, 1, False), (1, 45, 30000, 128, 64, 8, False),
                                                      (1, 13, 32768, 64, 16, 16, True), (1, 2, 118800, 64, 16, 1, False)])
def test_selection_without_scores_equals_selection_from_memory(B, H, L, d, M, N, tokens_first):
    rows, G = B * H * ((L + M - 1) // M), (L + N - 1) // N
    assert rows * G >= (72 if d == 128 else 48) << 20 and G >= 2048
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L + d)

    def tensor():
        x = torch.randn((B, L, H, d) if tokens_first else (B, H, L, d), generator=gen, device="cuda").bfloat16()
        return x.transpose(1, 2) if tokens_first else x
    q, k = tensor(), tensor()
    indptr = torch.empty(rows + 1, dtype=torch.int64, device="cuda")
    for kind, top_p, gain in (("spread", 0.3, 1.0), ("peaked", 0.9, 30.0), ("negative", 0.5, -4.0), ("crowded", 0.9, 1.0), ("every", 1.0, 4.0)):
        if kind == "crowded":
            q, k = q.abs(), k.clone()
            k[:, ::2] = 1.0 + (k[:, ::2] > 1.0).to(k.dtype) * 2.0 ** -7
            k[:, ::2, L // 2:L // 2 + N] = 40.0
        if kind == "every" and rows * G > 1 << 29:
            continue   # (ids of nearly all pairs)
        res = []
        for flags in (0, F.FLAG_MASK_ROWS_IN_HBM):
            p = F.make_params(q, k, k, q, M, N, gain * d ** -0.5, flags)
            ws = torch.empty(F.fgattn_mask_workspace_bytes(p), dtype=torch.uint8, device="cuda")
            F.fgattn_mask_select(q, k, p, top_p, indptr, ws)
            res.append((indptr.clone(), emitted(p, ws, indptr)))
        say("    %s: %.3f kept" % (kind, int(indptr[-1]) / (rows * G)))
        assert torch.equal(res[0][0], res[1][0]), kind
        assert torch.equal(res[0][1], res[1][1]), kind


# Rows short enough for a wave each: a lane's count of scores on both sides of every step, query blocks off a multiple of the
# workgroup's eight, key block means and K in place; scores spread out, without weight, equal, of few values (more than 64 members of
# the crossing bin) and crowded
@pytest.mark.parametrize("B,H,L,d,M,N", [(1, 3, 64, 64, 16, 1), (1, 2, 65, 128, 16, 1), (2, 2, 129, 64, 16, 1), (1, 2, 256, 128, 128, 1),
                                         (1, 3, 2050, 64, 32, 8), (1, 1, 512, 128, 16, 1), (2, 3, 8208, 128, 64, 16), (1, 2, 1023, 64, 16, 1),
                                         (1, 2, 1024, 128, 64, 1), (1, 2, 1025, 64, 64, 1)])
def test_short_rows_equal_selection_from_memory(B, H, L, d, M, N):
    rows, G = B * H * ((L + M - 1) // M), (L + N - 1) // N
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L + d)
    q, k0 = (torch.randn((B, H, L, d), generator=gen, device="cuda").bfloat16() for _ in range(2))
    indptr = torch.empty(rows + 1, dtype=torch.int64, device="cuda")
    for kind, gain in (("spread", 1.0), ("peaked", 30.0), ("negative", -4.0), ("equal", 1.0), ("few values", 1.0), ("crowded", 1.0), ("zero scale", 0.0)):
        k = k0
        if kind == "equal":
            k = torch.ones_like(k0)
        elif kind == "few values":
            k = (k0[..., :1] > 0.5).to(k0.dtype).expand_as(k0).contiguous()
        elif kind == "crowded":
            k = 1.0 + (k0 > 1.0).to(k0.dtype) * 2.0 ** -7
            k[:, :, L // 2:L // 2 + N] = 40.0
        for top_p in (0.3, 0.9, 1.0):
            res = []
            for flags in (0, F.FLAG_MASK_ROWS_IN_HBM):
                p = F.make_params(q, k, k, q, M, N, gain * d ** -0.5, flags)
                ws = torch.empty(F.fgattn_mask_workspace_bytes(p), dtype=torch.uint8, device="cuda")
                F.fgattn_mask_select(q, k, p, top_p, indptr, ws)
                res.append((indptr.clone(), emitted(p, ws, indptr)))
            assert torch.equal(res[0][0], res[1][0]), (kind, top_p)
            assert torch.equal(res[0][1], res[1][1]), (kind, top_p)


# Rows whose scores leave no usable range: equal scores (zero query blocks among ordinary ones, heads of identical keys), at scales
# above 1 that take the largest floats to infinity, scale zero, a range below the smallest one that can be divided by, and scores that
# are infinite.  No row stays empty, and a row of equal scores keeps its first ceil(p G) key blocks.
@pytest.mark.parametrize("H,L,d,M,N", [(1, 33000, 64, 16, 1), (3, 30001, 128, 32, 1), (5, 80000, 64, 64, 8), (3, 2047, 64, 32, 2), (2, 300, 128, 16, 1)])
def test_rows_without_a_range(H, L, d, M, N):
    QB, G = (L + M - 1) // M, (L + N - 1) // N
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    q0, k0 = (torch.nn.functional.normalize(torch.randn((1, H, L, d), generator=gen, device="cuda"), dim=-1).bfloat16() for _ in range(2))
    indptr = torch.empty(H * QB + 1, dtype=torch.int64, device="cuda")
    for kind, scale in (("zero blocks", 10.0), ("zero blocks", -4.0), ("identical keys", 1.5), ("identical keys", 4.0), ("identical keys", -64.0),
                        ("ordinary", 0.0), ("ordinary", 1e-38), ("infinite", 1.0), ("some infinite", 1.0)):
        q, k, equal = q0.clone(), k0.clone(), torch.zeros((H, QB), dtype=torch.bool, device="cuda")
        if kind == "zero blocks":
            equal[:, ::3] = True
            q[equal.repeat_interleave(M, 1)[None, :, :L]] = 0.0
        elif kind == "identical keys":
            equal[::2] = True
            k[:, ::2] = k[:, ::2, :1]
        elif "infinite" in kind:
            q, k = q.abs() * 2.0 ** 70, k.abs()
            k[:, :, ::97 if kind == "some infinite" else 1] *= 2.0 ** 70
        for top_p in (0.3, 0.9):
            res = []
            for flags in (0, F.FLAG_MASK_ROWS_IN_HBM):
                p = F.make_params(q, k, k, q, M, N, scale, flags)
                ws = torch.empty(F.fgattn_mask_workspace_bytes(p), dtype=torch.uint8, device="cuda")
                F.fgattn_mask_select(q, k, p, top_p, indptr, ws)
                res.append((indptr.clone(), emitted(p, ws, indptr)))
            say("    %s, scale %g: %d and %d kept" % (kind, scale, int(res[0][0][-1]), int(res[1][0][-1])))
            counts = (res[0][0][1:] - res[0][0][:-1]).view(H, QB)
            assert int(counts.min()) >= 1, (kind, scale)
            want = int(np.ceil(float(np.float32(top_p)) * G))
            assert (counts[equal] == want).all(), (kind, scale)
            first = torch.zeros((H * QB, G), dtype=torch.bool, device="cuda")
            first[torch.repeat_interleave(torch.arange(H * QB, device="cuda"), counts.view(-1)), res[0][1].long()] = True
            assert first.view(H, QB, G)[equal][:, :want].all(), (kind, scale)
            assert torch.equal(res[0][0], res[1][0]), (kind, scale)
            assert torch.equal(res[0][1], res[1][1]), (kind, scale)


# Long rows whose crossing bin holds more key blocks than the lists take: a few values (equal members), scores crowded beside a large
# negative one (several narrowings), half of them equal in the crowd (a single score left after narrowing, to be counted), most of
# them above or below those that come first and are listed, two scores one bit apart (scale zero).  Eight rows per workgroup and 32; stretches of the sweep that divide over the waves and that do not;
# some heads ordinary; row ends off a tile and a group of rows.
@pytest.mark.parametrize("H,L,d,M,N", [(1, 32000, 64, 16, 1), (1, 50001, 128, 32, 1), (1, 33000, 64, 16, 1), (3, 30001, 128, 32, 1), (6, 22000, 128, 32, 1),
                                       (66, 40000, 64, 128, 16)])
def test_long_rows_with_many_members(H, L, d, M, N):
    QB, G = (L + M - 1) // M, (L + N - 1) // N
    assert H * QB * G >= (72 if d == 128 else 48 if H * QB >= 2048 else 54) << 20 and H * QB >= 1024 and G >= 2048   # (or kept scores are taken)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    q0, k0 = (torch.randn((1, H, L, d), generator=gen, device="cuda").bfloat16() for _ in range(2))
    indptr = torch.empty(H * QB + 1, dtype=torch.int64, device="cuda")
    for kind, gain in (("two values", 1.0), ("few values", -1.0), ("crowded", 1.0), ("equal and crowded", 1.0), ("drifting and crowded", 1.0),
                       ("zero scale", 0.0)):
        q, k = q0, k0.clone()
        if kind == "two values":
            k[:] = (k0[..., :1] > 0.5).to(k0.dtype)
        elif kind == "few values":
            k[:] = (k0[..., :1].float().clamp(-1.2, 1.2) * 1.5).round().to(k0.dtype)
        elif "crowded" in kind:
            q = q0.abs()
            k = 1.0 + (k0 > 1.0).to(k0.dtype) * 2.0 ** -7
            if kind == "equal and crowded":
                k[:, :, (torch.arange(L, device="cuda") // N) % 2 == 0] = 1.0
            if kind == "drifting and crowded":   # the first fifth of every 512 key blocks in the middle of the others
                step = torch.randint(0, 18, (H, L), generator=gen, device="cuda")
                early = (torch.arange(L, device="cuda") // N) % 512 < 102
                k[0] = (1.0 + 2.0 ** -7 * torch.where(early, 8 + step % 2, step)).to(k0.dtype)[:, :, None]
            k[:, :, L // 2:L // 2 + N] = -40.0
        if H > 2:
            k[:, 1] = k0[:, 1]
        for top_p in (0.2, 0.9, 1.0) if H * QB * G < 1 << 27 else (0.9,):
            res = []
            for flags in (0, F.FLAG_MASK_ROWS_IN_HBM):
                p = F.make_params(q, k, k, q, M, N, gain * d ** -0.5, flags)
                ws = torch.empty(F.fgattn_mask_workspace_bytes(p), dtype=torch.uint8, device="cuda")
                F.fgattn_mask_select(q, k, p, top_p, indptr, ws)
                res.append((indptr.clone(), emitted(p, ws, indptr)))
            say("    %s, p %g: %d and %d kept" % (kind, top_p, int(res[0][0][-1]), int(res[1][0][-1])))
            assert torch.equal(res[0][0], res[1][0]), (kind, top_p)
            assert torch.equal(res[0][1], res[1][1]), (kind, top_p)


# So many query blocks that the sweep of all slices at once would make stretches longer than a list can count: chunks of fewer slices
def test_selection_without_scores_of_many_query_blocks():
    H, L, d, M = 96, 131072, 64, 128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    q, k = (torch.randn((1, H, L, d), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    indptr = torch.empty(H * L // M + 1, dtype=torch.int64, device="cuda")
    res = []
    for flags in (0, F.FLAG_MASK_ROWS_IN_HBM):
        p = F.make_params(q, k, k, q, M, 1, d ** -0.5, flags)
        ws = torch.empty(F.fgattn_mask_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        F.fgattn_mask_select(q, k, p, 0.02, indptr, ws)
        res.append((indptr.clone(), emitted(p, ws, indptr)))
    say("    %d and %d kept" % (int(res[0][0][-1]), int(res[1][0][-1])))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
