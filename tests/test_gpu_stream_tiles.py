"""GPU parity of both index streams at the edges of their units (4,096 entries) and
tiles (several units each past 4,095 units), with one segment, and with
segments that start late, in the middle of a unit, on a unit's edge and several
at one entry.  Encode against the oracle, decode back to the list, and the
workspace's table left zero."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_03839_amd import pulse
from tests.gpu_helpers import counter, dev, h32, read_count

pytestmark = pytest.mark.gpu

UNIT = 4096
SIZES = [1, 3, 4, 5, UNIT - 1, UNIT, UNIT + 1, 3 * UNIT + 2, 4095 * UNIT, 4095 * UNIT + 7]


def starts_for(n, how):
    if how == "one" or n < 3:
        return np.zeros(1, np.int64)
    if how == "late":  # entries before the first start belong to the list's start
        return np.array([n // 3], np.int64)
    s = [0, n // 7, n // 7, UNIT, UNIT, 2 * UNIT + 1, n // 2, n - 1, n, n + 3]
    return np.array(sorted(min(x, n) for x in s), np.int64)


def ascending(rng, n, segs, gap):
    idx = np.cumsum(rng.integers(1, 2 * gap, n, dtype=np.int64))
    bounds = [0] + [int(s) for s in segs if 0 < s < n]
    for b, e in zip(bounds, bounds[1:] + [n]):
        idx[b:e] -= idx[b] - int(rng.integers(0, gap))
    return idx.astype(np.uint32)


def split(idx, segs):
    b = sorted({0, *[int(s) for s in segs if s < idx.size]})
    return [idx[a:e] for a, e in zip(b, b[1:] + [idx.size])]


@pytest.mark.parametrize("how", ["one", "late", "many"])
@pytest.mark.parametrize("n", SIZES)
def test_varint_units_and_tiles(n, how):
    rng = np.random.default_rng(n + len(how))
    segs = starts_for(n, how)
    idx = ascending(rng, n, segs, 100 if n < 1 << 20 else 60)
    want = np.concatenate([oracle.varint_encode(x) for x in split(idx, segs)])
    ws = pulse.workspace()
    shift = 5  # the stream starts at an odd address
    out = torch.zeros(want.size + 64 + shift, dtype=torch.uint8, device="cuda")
    total, seg_d = counter(0), dev(segs)
    pulse.varint_encode(dev(idx), counter(n), out[shift:], total, ws, seg_begin=seg_d)
    torch.cuda.synchronize()
    assert read_count(total) == want.size
    np.testing.assert_array_equal(out[shift:shift + want.size].cpu().numpy(), want)
    back = torch.full((n + 3,), -1, dtype=torch.int32, device="cuda")
    got, stream = counter(0), dev(want)
    pulse.varint_decode(stream, counter(want.size), back, got, ws, seg_begin=seg_d)
    torch.cuda.synchronize()
    assert read_count(got) == n
    np.testing.assert_array_equal(h32(back)[:n], idx)
    assert (h32(back)[n:] == 0xFFFFFFFF).all()
    assert int(ws.view(torch.int64)[64:].abs().sum().item()) == 0


@pytest.mark.parametrize("how,cols", [("one", 1000), ("one", 3), ("many", 257), ("many", 65535)])
@pytest.mark.parametrize("n", SIZES)
def test_coo_units_and_tiles(n, how, cols):
    rng = np.random.default_rng(n + cols)
    segs = starts_for(n, how)
    idx = ascending(rng, n, segs, 60)
    c = np.full(segs.size, cols, np.uint32)
    of, od, oc, osp = oracle.coo_encode(idx, segs.astype(np.uint64), c)
    ws = pulse.workspace()
    drow = torch.zeros(od.size + 8, dtype=torch.uint8, device="cuda")
    dcol = torch.zeros(od.size + 8, dtype=torch.int16, device="cuda")
    first = torch.zeros(segs.size, dtype=torch.int32, device="cuda")
    sp = torch.zeros(segs.size, dtype=torch.int64, device="cuda")
    total, seg_d, cols_d = counter(0), dev(segs), dev(c)
    pulse.coo_encode(dev(idx), counter(n), seg_d, cols_d, first, drow, dcol, sp, total, ws)
    torch.cuda.synchronize()
    assert read_count(total) == od.size
    np.testing.assert_array_equal(drow[:od.size].cpu().numpy(), od)
    np.testing.assert_array_equal(dcol[:od.size].cpu().numpy().view(np.uint16), oc)
    np.testing.assert_array_equal(sp.cpu().numpy(), osp.astype(np.int64))
    np.testing.assert_array_equal(h32(first), of)
    back = torch.full((n + 3,), -1, dtype=torch.int32, device="cuda")
    pulse.coo_decode(drow, dcol, total, seg_d, sp, cols_d, first, counter(n), back, ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(h32(back)[:n], idx)
    assert (h32(back)[n:] == 0xFFFFFFFF).all()
    assert int(ws.view(torch.int64)[64:].abs().sum().item()) == 0


@pytest.mark.parametrize("nseg,most", [(300, 7), (3000, 7), (3000, 40), (2500, 3000)])
def test_varint_many_segments(nseg, most):
    """Segments of 0 to `most` entries, so that starts fall on every entry of a
    thread's quads, several at one entry, hundreds in a unit (past the 256 kept per
    tile) or several tiles apart, with numbers of one to four bytes: the stream, each
    segment's byte offset, and the list decoded back."""
    rng = np.random.default_rng(nseg + most)
    sizes = rng.integers(0, most + 1, nseg)
    segs = []
    for k in sizes:
        gap = np.exp2(rng.uniform(0, [6, 6, 13, 20][rng.integers(0, 4)] if most > 100 else 26, k)).astype(np.int64)
        segs.append(np.cumsum(gap).astype(np.uint32))
    begins = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    parts = [oracle.varint_encode(s) for s in segs]
    want, offs = np.concatenate(parts), np.concatenate([[0], np.cumsum([p.size for p in parts])[:-1]])
    idx, n = np.concatenate(segs), int(sizes.sum())
    ws, seg_d = pulse.workspace(), dev(begins)
    out = torch.zeros(want.size + 8, dtype=torch.uint8, device="cuda")
    total, at = counter(0), torch.full((nseg,), -1, dtype=torch.int64, device="cuda")
    pulse.varint_encode(dev(idx), counter(n), out, total, ws, seg_begin=seg_d, seg_bytes=at)
    torch.cuda.synchronize()
    assert read_count(total) == want.size
    np.testing.assert_array_equal(out[:want.size].cpu().numpy(), want)
    np.testing.assert_array_equal(at.cpu().numpy(), offs)
    back, got = torch.full((n + 3,), -1, dtype=torch.int32, device="cuda"), counter(0)
    pulse.varint_decode(out, total, back, got, ws, seg_begin=seg_d)
    torch.cuda.synchronize()
    assert read_count(got) == n
    np.testing.assert_array_equal(h32(back)[:n], idx)
    assert (h32(back)[n:] == 0xFFFFFFFF).all()


def test_streams_after_a_tensor_table():
    """One workspace for a batch whose descriptors lie in its table and for both
    streams: they write every word before they read it, so what the batch left
    there does not matter, and a batch after them finds its own."""
    rng = np.random.default_rng(77)
    ws = pulse.workspace()
    sizes = rng.integers(1, 5000, 300)
    w = [rng.standard_normal(n, dtype=np.float32) for n in sizes]
    s = [oracle.cast(x) ^ (rng.random(x.size) < 0.05).astype(np.uint16) for x in w]
    want = [oracle.encode(a, b) for a, b in zip(w, s)]
    o_idx = np.concatenate([i[:c] for c, i, _ in want])
    begins = np.concatenate([[0], np.cumsum([c for c, _, _ in want])[:-1]]).astype(np.int64)
    nnz = o_idx.size
    cols = np.minimum(sizes, 1000).astype(np.uint32)
    stream = np.concatenate([oracle.varint_encode(o_idx[a:a + c]) for a, (c, _, _) in zip(begins, want)])
    of, od, oc, osp = oracle.coo_encode(o_idx, begins.astype(np.uint64), cols)
    batch = pulse.EncodeBatch([pulse.EncodeTensor(dev(a), dev(b)) for a, b in zip(w, s)])
    for _ in range(3):
        idx = torch.zeros(nnz, dtype=torch.int32, device="cuda")
        val = torch.zeros(nnz, dtype=torch.int16, device="cuda")
        count, seg = counter(0), torch.full((sizes.size,), -1, dtype=torch.int64, device="cuda")
        batch(idx, val, count, ws, seg_begin=seg)
        out = torch.zeros(stream.size + 16, dtype=torch.uint8, device="cuda")
        total, got, back = counter(0), counter(0), torch.zeros(nnz, dtype=torch.int32, device="cuda")
        pulse.varint_encode(idx, count, out, total, ws, seg_begin=seg)
        batch(idx, val, counter(0), ws, seg_begin=seg)  # the table again, between encode and decode
        pulse.varint_decode(out, total, back, got, ws, seg_begin=seg)
        drow = torch.zeros(od.size, dtype=torch.uint8, device="cuda")
        dcol = torch.zeros(od.size, dtype=torch.int16, device="cuda")
        first = torch.zeros(sizes.size, dtype=torch.int32, device="cuda")
        sp, pairs, back2 = torch.zeros_like(seg), counter(0), torch.zeros_like(back)
        pulse.coo_encode(idx, count, seg, dev(cols), first, drow, dcol, sp, pairs, ws)
        batch(idx, val, counter(0), ws, seg_begin=seg)
        pulse.coo_decode(drow, dcol, pairs, seg, sp, dev(cols), first, count, back2, ws)
        torch.cuda.synchronize()
        assert read_count(count) == read_count(got) == nnz and read_count(total) == stream.size
        np.testing.assert_array_equal(seg.cpu().numpy(), begins)
        for i in (idx, back, back2):
            np.testing.assert_array_equal(h32(i), o_idx)
        np.testing.assert_array_equal(out[:stream.size].cpu().numpy(), stream)
        np.testing.assert_array_equal(drow.cpu().numpy(), od)
        np.testing.assert_array_equal(dcol.cpu().numpy().view(np.uint16), oc)
        np.testing.assert_array_equal(h32(first), of)
        np.testing.assert_array_equal(sp.cpu().numpy(), osp.astype(np.int64))
    pulse.check_workspace(ws)
