"""GPU parity of the small-call forms of the encoders and sparsifiers (one tile of
1, 2 or 4 groups of 8,192 elements per block), at the edges of their tiles and
at the sizes where a call leaves one form for the next, and of the persistent
form at the same edges (beside a tensor large enough to select it).  Against
the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_03839_amd import pulse
from tests.gpu_helpers import counter, dev, h16, h32, hf32, read_count

pytestmark = pytest.mark.gpu

G = 8192
# last size of each form and the first of the next; a form's tile edges
EDGES = [1, G - 1, G, G + 1, 3 * G + 5, 128 * G, 128 * G + 1, 130 * G + 2 * G - 1, 256 * 2 * G, 256 * 2 * G + 1,
         300 * 2 * G + 4 * G + 9]
LAST = 512 * 4 * G      # the encoders' last one-tile size
LAST_LOCO = 768 * G     # the sparsifiers'
SMALL = [1, 7, 8, 9, 511, 512, 513, 7679, 7680, 7681, 15359, 15360, 15361, 23041]


@pytest.fixture(scope="module")
def ws():
    return pulse.workspace()


def encode_check(ws, sizes, density, cap_frac, count_in=0):
    rng = np.random.default_rng(sum(sizes) * 3 + len(sizes) + int(density * 100))
    host, descs, base = [], [], 0
    for n in sizes:
        w = rng.standard_normal(n, dtype=np.float32)
        s = oracle.cast(w) ^ (rng.random(n, dtype=np.float32) < density).astype(np.uint16)
        s_d = dev(s)
        host.append((w, s, base))
        descs.append(pulse.EncodeTensor(dev(w), s_d, s_d.clone(), base, mirrors_snap=True))
        base += n
    nnz = sum(int((oracle.cast(w) != s).sum()) for w, s, _ in host)
    cap = count_in + int(nnz * cap_frac)
    o_idx, o_val, o_seg, cnt = np.zeros(max(cap, 1), np.uint32), np.zeros(max(cap, 1), np.uint16), [], count_in
    o_refs = []
    for w, s, b in host:
        o_seg.append(cnt)
        r = s.copy()
        cnt, _, _ = oracle.encode(w, s, index_base=b, capacity=cap, count_in=cnt, idx_out=o_idx,
                                  val_out=o_val, refresh=r)
        o_refs.append(r)
    # the plain form, then the mirrored one
    plain = [pulse.EncodeTensor(d.w_new, d.snap, None, d.index_base) for d in descs]
    for batch in (plain, descs):
        idx = torch.zeros(max(cap, 1), dtype=torch.int32, device="cuda")
        val = torch.zeros(max(cap, 1), dtype=torch.int16, device="cuda")
        count, seg = counter(count_in), torch.full((len(sizes),), -1, dtype=torch.int64, device="cuda")
        pulse.EncodeBatch(batch)(idx, val, count, ws, seg_begin=seg, capacity=cap)
        torch.cuda.synchronize()
        assert read_count(count) == cnt
        np.testing.assert_array_equal(seg.cpu().numpy(), np.array(o_seg))
        m = min(cnt, cap)
        np.testing.assert_array_equal(h32(idx)[count_in:m], o_idx[count_in:m])
        np.testing.assert_array_equal(h16(val)[count_in:m], o_val[count_in:m])
    for d, r in zip(descs, o_refs):
        np.testing.assert_array_equal(h16(d.refresh), r)
    pulse.check_workspace(ws)


@pytest.mark.parametrize("n", EDGES)
@pytest.mark.parametrize("density,cap_frac", [(0.01, 1.0), (0.4, 0.5)])
def test_encode_one_tile_edges(ws, n, density, cap_frac):
    encode_check(ws, [n], density, cap_frac, count_in=5)


@pytest.mark.parametrize("n", [LAST, LAST + 1])
def test_encode_last_one_tile_size(ws, n):
    encode_check(ws, [n], 0.01, 1.0)


@pytest.mark.parametrize("big", [0, LAST + 1])
@pytest.mark.parametrize("cap_frac", [1.0, 0.7])
def test_encode_ragged_batch_both_forms(ws, big, cap_frac):
    encode_check(ws, SMALL + ([big] if big else []) + SMALL[::-1], 0.3, cap_frac)


def loco_check(ws, sizes, theta, tau, cap_frac):
    rng = np.random.default_rng(sum(sizes) + len(sizes))
    descs, want, o_seg, cnt, base = [], [], [], 0, 0
    N = sum(sizes)
    host = []
    for n in sizes:
        th = (0.1 * rng.standard_normal(n, dtype=np.float32)) if theta else None
        host.append((2e-4 * rng.standard_normal(n, dtype=np.float32),
                     5e-5 * rng.standard_normal(n, dtype=np.float32), th))
    cap = int(N * cap_frac)
    o_idx, o_val = np.zeros(N, np.uint32), np.zeros(N, np.float32)
    for (d, e, th), n in zip(host, sizes):
        e_d = dev(e)
        descs.append(pulse.LocoTensor(dev(d), e_d, dev(th) if theta else None, base))
        o_seg.append(cnt)
        k, oi, ov = oracle.loco(d, e, tau, theta=th, index_base=base, capacity=max(0, cap - cnt))
        sent = min(k, max(0, cap - cnt))
        o_idx[cnt:cnt + sent], o_val[cnt:cnt + sent] = oi[:sent], ov[:sent]
        cnt += k
        want.append((e_d, e))
        base += n
    idx = torch.zeros(max(cap, 1), dtype=torch.int32, device="cuda")
    val = torch.zeros(max(cap, 1), dtype=torch.float32, device="cuda")
    count, seg = counter(0), torch.full((len(sizes),), -1, dtype=torch.int64, device="cuda")
    pulse.LocoBatch(descs)(tau, idx, val, count, ws, seg_begin=seg, capacity=cap)
    torch.cuda.synchronize()
    assert read_count(count) == cnt
    np.testing.assert_array_equal(seg.cpu().numpy(), np.array(o_seg))
    m = min(cnt, cap)
    np.testing.assert_array_equal(h32(idx)[:m], o_idx[:m])
    np.testing.assert_array_equal(hf32(val)[:m].view(np.uint32), o_val[:m].view(np.uint32))
    for e_d, e in want:
        np.testing.assert_array_equal(hf32(e_d).view(np.uint32), e.view(np.uint32))
    pulse.check_workspace(ws)


@pytest.mark.parametrize("theta", [False, True])
@pytest.mark.parametrize("cap_frac", [1.0, 0.01])
@pytest.mark.parametrize("sizes", [[G - 1], [G + 1], [LAST_LOCO], [LAST_LOCO + 1], SMALL, SMALL + [LAST_LOCO + 1] + SMALL],
                         ids=["G-1", "G+1", "last", "last+1", "ragged", "ragged_persistent"])
def test_loco_one_tile_and_persistent(ws, theta, cap_frac, sizes):
    loco_check(ws, sizes, theta, 3e-4, cap_frac)


@pytest.mark.parametrize("dtype", [pulse.FP8_E4M3, pulse.MXFP4])
@pytest.mark.parametrize("sizes", [[n] for n in EDGES] + [SMALL, SMALL + [LAST + 1] + SMALL], ids=lambda s: "%dx%d" % (len(s), max(s)))
def test_lowp_one_tile_and_persistent(ws, dtype, sizes):
    rng = np.random.default_rng(sum(sizes) + dtype)
    fp8 = dtype == pulse.FP8_E4M3
    descs, o_seg, o_idx, o_val, cnt = [], [], [], [], 0
    for n in sizes:
        w = 0.1 * rng.standard_normal(n, dtype=np.float32)
        w2 = w + 1e-3 * rng.standard_normal(n, dtype=np.float32)
        o_seg.append(cnt)
        if fp8:
            snap, sc = oracle.cast_fp8(w, 900.0), None
            k, oi, ov = oracle.encode_fp8(w2, snap, 900.0)
        else:
            snap, sc = oracle.cast_mxfp4(w)
            k, oi, ov = oracle.encode_mxfp4(w2, snap, sc)
        o_idx.append(oi[:k].copy())
        o_val.append(ov[:k].copy())
        cnt += k
        descs.append(pulse.LowpTensor(dev(w2), dev(snap), None if fp8 else dev(sc), 0, 900.0))
    idx = torch.zeros(max(cnt, 1), dtype=torch.int32, device="cuda")
    val = torch.zeros(max(cnt, 1), dtype=torch.uint8 if fp8 else torch.int16, device="cuda")
    count, seg = counter(0), torch.full((len(sizes),), -1, dtype=torch.int64, device="cuda")
    pulse.EncodeLowpBatch(dtype, descs)(idx, val, count, ws, seg_begin=seg)
    torch.cuda.synchronize()
    assert read_count(count) == cnt
    np.testing.assert_array_equal(seg.cpu().numpy(), np.array(o_seg))
    np.testing.assert_array_equal(h32(idx)[:cnt], np.concatenate(o_idx))
    got = val.cpu().numpy() if fp8 else h16(val)
    np.testing.assert_array_equal(got[:cnt], np.concatenate(o_val))
    pulse.check_workspace(ws)


# Many tensors with ragged ends in the four-group form, past 256 blocks: every
# length modulo 8 (and modulo the 32 values of an MXFP4 block), ends at and beside
# the edges of groups, waves and tiles, and tensors of less than one lane's load.
RAGGED4 = [4 * G * (3 + i) + [0, 1, 7, 8, 9, 511, G - 1, G, G + 1, 2 * G + 25, 3 * G + 3][i % 11] + 13 * i
           for i in range(22)] + [n for n in range(1, 18)] + [31, 32, 33, 4 * G, 4 * G - 1]


def test_ragged4_takes_the_four_group_form():
    tiles = [sum(-(-n // (g * G)) for n in RAGGED4) for g in (1, 2, 4)]
    assert tiles[0] > 128 and tiles[1] > 256 and 256 < tiles[2] <= 512


@pytest.mark.parametrize("density,cap_frac", [(0.01, 1.0), (0.3, 0.6)])
def test_encode_many_ragged_tensors_four_groups(ws, density, cap_frac):
    encode_check(ws, RAGGED4, density, cap_frac, count_in=3)


@pytest.mark.parametrize("dtype", [pulse.FP8_E4M3, pulse.MXFP4])
def test_lowp_many_ragged_tensors_four_groups(ws, dtype):
    test_lowp_one_tile_and_persistent(ws, dtype, RAGGED4)


@pytest.mark.parametrize("tiles,ragged", [((1 << 16) - 1, 0), (1 << 16, 5), ((1 << 16) + 3, 0)])
@pytest.mark.parametrize("refresh", [False, True])
def test_encode_tiles_per_ticket(ws, tiles, ragged, refresh):
    """The persistent encode around the launch size where the form without refresh
    takes four tiles per ticket instead of two: masters and snapshot zero but for
    2M places whose patch the host knows, clustered in some tiles."""
    n = tiles * 15360 - ragged
    rng = np.random.default_rng(tiles + ragged)
    at = np.unique(np.concatenate([rng.integers(0, n, 1_500_000), rng.integers(n // 2, n // 2 + 900_000, 500_000),
                                   np.arange(n - 300, n), np.arange(300)]))
    v = rng.standard_normal(at.size, dtype=np.float32)
    bits = oracle.cast(v)
    w = torch.zeros(n, dtype=torch.float32, device="cuda")
    w[torch.from_numpy(at).cuda()] = dev(v)
    snap = torch.zeros(n, dtype=torch.int16, device="cuda")
    keep = bits != 0
    at, bits = at[keep], bits[keep]
    idx = torch.zeros(at.size + 5, dtype=torch.int32, device="cuda")
    val = torch.zeros(at.size + 5, dtype=torch.int16, device="cuda")
    copy = torch.zeros(n, dtype=torch.int16, device="cuda") if refresh else None
    count = counter(2)
    pulse.encode(w, snap, idx, val, count, ws, refresh=copy)
    torch.cuda.synchronize()
    assert read_count(count) == at.size + 2
    np.testing.assert_array_equal(h32(idx)[2:-3], at.astype(np.uint32))
    np.testing.assert_array_equal(h16(val)[2:-3], bits)
    if refresh:
        assert int((copy != 0).sum().item()) == at.size
        np.testing.assert_array_equal(h16(copy[torch.from_numpy(at).cuda()]), bits)
    pulse.check_workspace(ws)
