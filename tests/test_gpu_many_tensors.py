"""GPU parity of batches with more tensors than a launch's kernel arguments hold
(64): their descriptors go through the workspace's table, up to 1,024 tensors a
launch.  Encode (plain, mirrored, with the patch overflowing), the gate
sparsifier and the FP8/MXFP4 encodes against the oracle tensor by tensor, bit
for bit; the numbers of tensors sit at the table's edges."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_03839_amd import pulse
from tests.gpu_helpers import counter, dev, h16, h32, hf32, read_count

pytestmark = pytest.mark.gpu

COUNTS = [64, 65, 129, 1024, 1025, 1100]


def make_sizes(rng, T, big):
    """Mostly tiny and some empty tensors, a few of `big` elements and more, empty ones at both ends."""
    sizes = rng.integers(0, 60, T)
    sizes[rng.random(T) < 0.2] = 0
    for at in (T // 3, T // 2, T - 2):
        sizes[at] = big + int(rng.integers(0, 100))
    sizes[0] = sizes[-1] = 0
    return [int(x) for x in sizes]


def f32(a):
    return dev(a) if a.size else torch.empty(0, dtype=torch.float32, device="cuda")


def i16(a):
    return dev(a) if a.size else torch.empty(0, dtype=torch.int16, device="cuda")


@pytest.fixture(scope="module")
def ws():
    return pulse.workspace()


def buffers(cap, T, val_dtype):
    return (torch.zeros(max(cap, 1), dtype=torch.int32, device="cuda"),
            torch.zeros(max(cap, 1), dtype=val_dtype, device="cuda"), counter(0),
            torch.full((T,), -1, dtype=torch.int64, device="cuda"))


@pytest.mark.parametrize("cap_frac", [None, 1.0, 0.5])
@pytest.mark.parametrize("T", COUNTS)
def test_encode_many_tensors(ws, T, cap_frac):
    """cap_frac None: no refresh; else mirrored refresh with that share of the patch's room."""
    rng = np.random.default_rng(T)
    sizes = make_sizes(rng, T, 40_000)
    host, descs, refs, base = [], [], [], 0
    for n in sizes:
        w = rng.normal(0, 0.1, n).astype(np.float32)
        s = oracle.cast(w) ^ (rng.random(n) < 0.03).astype(np.uint16)
        s_d = i16(s)
        r_d = s_d.clone() if cap_frac is not None else None
        host.append((w, s, base))
        refs.append(r_d)
        descs.append(pulse.EncodeTensor(f32(w), s_d, r_d, base, mirrors_snap=r_d is not None))
        base += n
    nnz = sum(int((oracle.cast(w) != s).sum()) for w, s, _ in host)
    cap = nnz if cap_frac is None else int(nnz * cap_frac)
    o_idx, o_val, o_seg, cnt = np.zeros(cap, np.uint32), np.zeros(cap, np.uint16), [], 0
    o_refs = []
    for w, s, b in host:
        o_seg.append(cnt)
        r = s.copy()
        cnt, _, _ = oracle.encode(w, s, index_base=b, capacity=cap, count_in=cnt, idx_out=o_idx,
                                  val_out=o_val, refresh=r)
        o_refs.append(r)
    idx, val, count, seg = buffers(cap, T, torch.int16)
    pulse.EncodeBatch(descs)(idx, val, count, ws, seg_begin=seg, capacity=cap)
    torch.cuda.synchronize()
    assert read_count(count) == cnt == nnz
    np.testing.assert_array_equal(seg.cpu().numpy(), np.array(o_seg))
    np.testing.assert_array_equal(h32(idx)[:cap], o_idx)
    np.testing.assert_array_equal(h16(val)[:cap], o_val)
    for t, (r_d, r) in enumerate(zip(refs, o_refs)):
        if r_d is not None and r.size:
            np.testing.assert_array_equal(h16(r_d), r, err_msg=str(t))
    pulse.check_workspace(ws)


@pytest.mark.parametrize("T", COUNTS)
def test_gate_many_tensors(ws, T):
    rng = np.random.default_rng(T + 1)
    sizes = make_sizes(rng, T, 20_000)
    descs, res, want, o_seg, cnt = [], [], [], [], 0
    cap = sum(sizes)
    o_idx, o_val = np.zeros(cap, np.uint32), np.zeros(cap, np.float32)
    for n in sizes:
        th = rng.normal(0, 0.1, n).astype(np.float32)
        d = rng.normal(0, 2e-4, n).astype(np.float32)
        e = rng.normal(0, 5e-5, n).astype(np.float32)
        e_d = f32(e)
        descs.append(pulse.LocoTensor(f32(d), e_d, f32(th), 0))
        o_seg.append(cnt)
        if n:
            k, oi, ov = oracle.loco(d, e, 0.0, theta=th)
            o_idx[cnt:cnt + k], o_val[cnt:cnt + k] = oi[:k], ov[:k]
            cnt += k
        res.append(e_d)
        want.append(e)
    idx, val, count, seg = buffers(cap, T, torch.float32)
    pulse.LocoBatch(descs)(0.0, idx, val, count, ws, seg_begin=seg)
    torch.cuda.synchronize()
    assert read_count(count) == cnt
    np.testing.assert_array_equal(seg.cpu().numpy(), np.array(o_seg))
    np.testing.assert_array_equal(h32(idx)[:cnt], o_idx[:cnt])
    np.testing.assert_array_equal(hf32(val)[:cnt].view(np.uint32), o_val[:cnt].view(np.uint32))
    for t, (r_d, r) in enumerate(zip(res, want)):
        np.testing.assert_array_equal(hf32(r_d).view(np.uint32), r.view(np.uint32), err_msg=str(t))


@pytest.mark.parametrize("dtype", [pulse.FP8_E4M3, pulse.MXFP4])
@pytest.mark.parametrize("T", COUNTS)
def test_lowp_many_tensors(ws, T, dtype):
    rng = np.random.default_rng(T + 2)
    fp8 = dtype == pulse.FP8_E4M3
    sizes = make_sizes(rng, T, 50_000)
    descs, o_seg, cnt = [], [], 0
    cap = sum(sizes)
    o_idx, o_val = np.zeros(cap, np.uint32), np.zeros(cap, np.uint8 if fp8 else np.uint16)
    for t, n in enumerate(sizes):
        w = rng.normal(0, 0.1, n).astype(np.float32)
        w2 = (w + rng.normal(0, 1e-3, n)).astype(np.float32)
        scale = 100.0 + t
        o_seg.append(cnt)
        if fp8:
            snap, sc = oracle.cast_fp8(w, scale), None
            k, oi, ov = oracle.encode_fp8(w2, snap, scale) if n else (0, o_idx, o_val)
        else:
            snap, sc = oracle.cast_mxfp4(w) if n else (np.zeros(0, np.uint8), np.zeros(0, np.uint8))
            k, oi, ov = oracle.encode_mxfp4(w2, snap, sc) if n else (0, o_idx, o_val)
        o_idx[cnt:cnt + k], o_val[cnt:cnt + k] = oi[:k], ov[:k]
        cnt += k
        u8 = lambda a: dev(a) if a.size else torch.empty(0, dtype=torch.uint8, device="cuda")  # noqa: E731
        descs.append(pulse.LowpTensor(f32(w2), u8(snap), None if fp8 else u8(sc), 0, scale))
    idx, val, count, seg = buffers(cap, T, torch.uint8 if fp8 else torch.int16)
    pulse.EncodeLowpBatch(dtype, descs)(idx, val, count, ws, seg_begin=seg)
    torch.cuda.synchronize()
    assert read_count(count) == cnt
    np.testing.assert_array_equal(seg.cpu().numpy(), np.array(o_seg))
    np.testing.assert_array_equal(h32(idx)[:cnt], o_idx[:cnt])
    got = val.cpu().numpy() if fp8 else h16(val)
    np.testing.assert_array_equal(got[:cnt], o_val[:cnt])


@pytest.mark.parametrize("T", [130, 1030])
def test_all_empty_many_tensors(ws, T):
    """No elements at all: every segment starts at the append position."""
    e = torch.empty(0, dtype=torch.float32, device="cuda")
    s = torch.empty(0, dtype=torch.int16, device="cuda")
    idx, val, count, seg = buffers(4, T, torch.int16)
    count.fill_(3)
    pulse.EncodeBatch([pulse.EncodeTensor(e, s)] * T)(idx, val, count, ws, seg_begin=seg)
    torch.cuda.synchronize()
    assert read_count(count) == 3
    assert bool((seg == 3).all())


@pytest.mark.parametrize("dtype", [None, pulse.FP8_E4M3, pulse.MXFP4])
@pytest.mark.parametrize("T", [1, 159, 160, 161, 223, 224, 225, 449])
def test_apply_many_tensors(T, dtype):
    """BF16, FP8 and MXFP4 applies at the edges of a launch's tensors, empty ones
    among them, entries outside their tensor counted and left out."""
    rng = np.random.default_rng(T + 3)
    sizes = [int(x) for x in rng.integers(0, 90, T)]
    sizes[0] = 5000
    idx, seg, at = [], [], 0
    for n in sizes:
        k = int(rng.integers(0, n + 1)) if n else 0
        i = np.sort(rng.choice(n, k, replace=False)) if k else np.zeros(0, np.int64)
        if rng.random() < 0.2:
            i = np.append(i, n + 3)  # outside
        idx.append(i.astype(np.uint32))
        seg.append(at)
        at += i.size
    all_idx = np.concatenate(idx)
    u8 = lambda a: dev(a) if a.size else torch.empty(0, dtype=torch.uint8, device="cuda")  # noqa: E731
    bad = sum(int((i >= n).sum()) for i, n in zip(idx, sizes))
    rej, end, seg_d = counter(0), counter(at), dev(np.array(seg, np.int64))
    if dtype is None:
        val = rng.integers(0, 1 << 16, at, dtype=np.uint16)
        host = [rng.integers(0, 1 << 16, n, dtype=np.uint16) for n in sizes]
        dst = [i16(h) for h in host]
        pulse.ApplyBatch([pulse.ApplyTensor(d) for d in dst])(dev(all_idx), dev(val), seg_d, end, rejected=rej)
        for t, (h, i, s) in enumerate(zip(host, idx, seg)):
            ok = i < h.size
            h[i[ok]] = val[s:s + i.size][ok]
            np.testing.assert_array_equal(h16(dst[t]), h, err_msg=str(t))
    else:
        fp8 = dtype == pulse.FP8_E4M3
        val = rng.integers(0, 256, at, dtype=np.uint8) if fp8 else \
            ((7 << 8) | rng.integers(0, 16, at)).astype(np.uint16)
        sz = [pulse.lowp_sizes(dtype, n) for n in sizes]
        codes = [rng.integers(0, 256, a, dtype=np.uint8) for a, _ in sz]
        scales = [rng.integers(0, 256, b, dtype=np.uint8) for _, b in sz]
        cd, sd = [u8(c) for c in codes], [u8(s) for s in scales]
        pulse.ApplyLowpBatch(dtype, [pulse.LowpApplyTensor(cd[t], None if fp8 else sd[t], n)
                                     for t, n in enumerate(sizes)])(dev(all_idx), dev(val), seg_d, end, rejected=rej)
        for t, (i, s, n) in enumerate(zip(idx, seg, sizes)):
            for j, v in zip(i, val[s:s + i.size]):
                if j >= n:
                    continue
                if fp8:
                    codes[t][j] = v
                else:
                    b = codes[t][j // 2]
                    codes[t][j // 2] = (b & 0x0F) | ((v & 0xF) << 4) if j & 1 else (b & 0xF0) | (v & 0xF)
                    scales[t][j // 32] = v >> 8
            np.testing.assert_array_equal(cd[t].cpu().numpy(), codes[t], err_msg=str(t))
            np.testing.assert_array_equal(sd[t].cpu().numpy(), scales[t], err_msg=str(t))
    assert read_count(rej) == bad


@pytest.mark.parametrize("T", [1024, 1025, 1100])
@pytest.mark.parametrize("cap_frac", [1.0, 0.3])
def test_threshold_two_pass_many_tensors(T, cap_frac):
    """The two-pass threshold form over more tensors than kernel arguments hold,
    with dense tiles that overflow their staging and entries past the capacity."""
    rng = np.random.default_rng(T + 4)
    sizes = make_sizes(rng, T, 30_000)
    N, tau = sum(sizes), 3e-4
    ws = pulse.loco_workspace(N)
    descs, res, want, o_seg, cnt = [], [], [], [], 0
    o_idx, o_val = np.zeros(N, np.uint32), np.zeros(N, np.float32)
    host = [(rng.normal(0, 2e-4, n).astype(np.float32), rng.normal(0, 5e-5, n).astype(np.float32)) for n in sizes]
    nnz = sum(int((np.abs(d + e) >= np.float32(tau)).sum()) for d, e in host)
    cap = int(nnz * cap_frac)
    for d, e in host:
        e_d = f32(e)
        descs.append(pulse.LocoTensor(f32(d), e_d, None, 0))
        o_seg.append(cnt)
        if d.size:
            room = max(0, cap - cnt)
            k, oi, ov = oracle.loco(d, e, tau, capacity=room)
            o_idx[cnt:cnt + min(k, room)], o_val[cnt:cnt + min(k, room)] = oi[:min(k, room)], ov[:min(k, room)]
            cnt += k
        res.append(e_d)
        want.append(e)
    idx, val, count, seg = buffers(cap, T, torch.float32)
    pulse.LocoBatch(descs)(tau, idx, val, count, ws, seg_begin=seg, capacity=cap)
    torch.cuda.synchronize()
    assert read_count(count) == cnt == nnz
    np.testing.assert_array_equal(seg.cpu().numpy(), np.array(o_seg))
    np.testing.assert_array_equal(h32(idx)[:cap], o_idx[:cap])
    np.testing.assert_array_equal(hf32(val)[:cap].view(np.uint32), o_val[:cap].view(np.uint32))
    for t, (r_d, r) in enumerate(zip(res, want)):
        np.testing.assert_array_equal(hf32(r_d).view(np.uint32), r.view(np.uint32), err_msg=str(t))


@pytest.mark.parametrize("capacity", [1, 255, 257, 2048 * 256 - 1, 2048 * 256 + 1, 2048 * 1024 + 5, 8192 * 1024 - 1,
                                      8192 * 1024 + 3])
def test_apply_capacity_sets_the_grid(capacity):
    """Each size of an apply's grid, with the entries at the capacity's end and
    more of them than one pass of the blocks takes."""
    rng = np.random.default_rng(capacity)
    k = min(capacity, 3_000_000)
    n = 4 * k + 9
    at = np.sort(rng.choice(n, k, replace=False)).astype(np.uint32)
    dst = rng.integers(0, 1 << 16, n).astype(np.uint16)
    idx = np.zeros(capacity, np.uint32)
    val = np.zeros(capacity, np.uint16)
    idx[capacity - k:], val[capacity - k:] = at, rng.integers(0, 1 << 16, k)
    dst_d, rejected = dev(dst), counter(0)
    pulse.apply(dst_d, dev(idx), dev(val), counter(capacity - k), counter(capacity + 10), rejected=rejected)
    torch.cuda.synchronize()
    dst[at] = val[capacity - k:]
    np.testing.assert_array_equal(h16(dst_d), dst)
    assert read_count(rejected) == 0
