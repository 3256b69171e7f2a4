"""CPU model of the addresses of the many-row LM-head kernel (csrc/lmhead_wide.hip:
workgroup -> tile mapping, Stream::init, load, request, zero_tail, the ring positions, the
fragment reads and the untruncated epilogue's dense rows): for every row shape, wave, lane, load and stage, global accesses stay inside
their operand, 32-bit lane offsets are exact, LDS accesses stay inside a stage, the loads
fill a stage, each fragment read finds the column the swizzle put there, no stage is filled
while a wave may still read it, and each is waited for before it is read."""
import numpy as np
import pytest

TT, CB, WL, KSTEP = 256, 128, 8, 64
LANE = np.arange(64)
SHAPES = range(4, 10)  # row blocks per wave


def _geo(rb):
    return dict(TR=32 * rb, HI=2 * rb, HL=(2 * rb + 3) // 4, HS=32 * rb * KSTEP,
                NW=4 if rb <= 4 else 3, NH=4 if 4 < rb <= 7 else 3)


def _tiles(R, V, TR):
    ntiles, nrt = (V + TT - 1) // TT, (R + TR - 1) // TR
    for gid in range((ntiles + 7) // 8 * 8 * nrt):
        xcd, local = gid % 8, gid // 8
        tile = local // nrt * 8 + xcd
        if tile < ntiles:
            yield tile, local % nrt * TR


def _lanes(half, wv, rb):
    """[(operand row in the tile, column byte, LDS byte in the stage)] of one wave's loads."""
    g = _geo(rb)
    out = []
    if half == 0:
        r, col = LANE // 8, ((LANE % 8) ^ (LANE // 8)) * 16
        for q in range(WL):
            out.append((64 * wv + 8 * q + r, col, 64 * wv * CB + q * 8 * CB + LANE * 16))
    else:
        r, col = LANE // 4, ((LANE % 4) ^ (-(LANE // 16) & 3)) * 16
        for k in range(g["HL"]):
            grp = min(wv + 4 * k, g["HI"] - 1)
            step = (k * 4 if k + 1 < g["HL"] else grp - wv) * 16 * KSTEP
            out.append((16 * grp + r, col, 16 * wv * KSTEP + step + LANE * 16))
    return out


@pytest.mark.parametrize("rb", SHAPES)
@pytest.mark.parametrize("R,V,d", [(65, 300, 8), (65, 257, 24), (129, 1000, 64), (129, 600, 72),
                                   (285, 4099, 200), (513, 5, 512), (651, 2500, 192), (2049, 1023, 256)])
def test_global_addresses_stay_in_bounds(R, V, d, rb):
    g, rowbytes = _geo(rb), 2 * d
    nch = (rowbytes + CB - 1) // CB
    seen = set()
    for tile, row0 in _tiles(R, V, g["TR"]):
        rot = nch - 1 if rowbytes % CB else (7 * tile % nch if R <= g["TR"] else 0)
        key = (min(V - tile * TT, TT), min(R - row0, g["TR"]), rot)
        if key in seen:
            continue
        seen.add(key)

        def koff(c):
            return (c + rot if c + rot < nch else c + rot - nch) * CB

        assert sorted(koff(c) for c in range(nch)) == [CB * c for c in range(nch)]
        for half, count, base in ((0, V, tile * TT), (1, R, row0)):
            stages = g["NW"] if half == 0 else g["NH"]
            per = 1 if half == 0 else 2  # stages per chunk
            for wv in range(4):
                for row, col, _ in _lanes(half, wv, rb):
                    c16 = np.minimum(col, rowbytes - 16)
                    off = np.minimum(row, count - 1 - base) * rowbytes + c16
                    for i in range(per * nch + stages + 2):
                        c = i // per
                        first = i < per
                        if half == 0:
                            k0 = koff(i if first else min(i, nch - 1))
                        else:
                            k0 = koff(c) + (i & 1) * KSTEP if c < nch else koff(nch - 1)
                        o = off
                        if first:
                            end = rowbytes - 16
                            at = np.minimum(k0 + col, end)
                            k0s, k0 = k0, min(k0, end)
                            o = off + (at - k0 - c16)
                        assert np.all(o >= 0) and np.all(o < 2 ** 32)
                        a = base * rowbytes + k0 + o
                        assert np.all(a >= 0) and np.all(a + 16 <= count * rowbytes)
                        if c < nch:  # a lane inside the row reads its own column
                            k0 = k0s if first else k0
                            ok = k0 + col < rowbytes
                            want = (base + np.minimum(row, count - 1 - base)) * rowbytes + k0 + col
                            assert np.array_equal(a[ok], want[ok])
                            assert first or ok.all()
    assert seen


@pytest.mark.parametrize("rb", SHAPES)
def test_stages_are_filled_and_read_where_they_were_put(rb):
    g = _geo(rb)
    w, h = np.full(TT * 8, -1, np.int64), np.full(g["TR"] * 4, -1, np.int64)
    for half, stage, cols in ((0, w, 8), (1, h, 4)):
        for wv in range(4):
            for row, col, at in _lanes(half, wv, rb):
                put = row * cols + col // 16
                assert np.all((stage[at // 16] == -1) | (stage[at // 16] == put))
                stage[at // 16] = put
        assert np.all(stage >= 0)
    n, k = LANE % 16, LANE // 16
    for wave in range(8):
        wt, G = wave % 4, wave // 4
        for s in range(2):
            wl = ((wt * 64 + n) * CB + (k ^ (n % 8)) * 16) ^ (KSTEP * s)
            for vb in range(4):
                assert np.array_equal(w[(wl + 2048 * vb) // 16], (wt * 64 + 16 * vb + n) * 8 + 4 * s + k)
        hl = (G * 16 * rb + n) * KSTEP + (k ^ (-(n // 4) & 3)) * 16
        for at, pitch in ((wl, CB), (hl, KSTEP)):  # the lane groups ds_read_b128 serves together
            for grp in ([0, 1, 2, 3, 12, 13, 14, 15] + list(range(20, 28)),
                        list(range(4, 12)) + [16, 17, 18, 19, 28, 29, 30, 31]):
                for half in (0, 32):
                    assert len(set(at[np.array(grp) + half] // 16 % 16)) == 16, pitch
        for b in range(rb):
            assert np.array_equal(h[(hl + 1024 * b) // 16], (G * 16 * rb + 16 * b + n) * 4 + k)


@pytest.mark.parametrize("rb", SHAPES)
@pytest.mark.parametrize("nch", [1, 2, 3, 4, 7])
def test_ring_schedule(rb, nch):
    """Slot by slot: requests never hit a stage that a read of the same or a later slot may
    use, the waits (in-order completion, the counts of run_pass) cover a stage before its
    first read, and both halves end the same number of slots."""
    g = _geo(rb)
    NW, NH = g["NW"], g["NH"]
    reads, fills, landed = {}, {}, {}
    # G = 0
    issued = list(range(NW - 1))
    for i in issued:
        landed[("w", i)] = -1  # wait_loads<0> before slot 0
    for c in range(nch):
        i = c + NW - 1
        fills[("w", i)] = (4 * c + 1, i % NW)  # (its second half in slot 4c+3)
        issued.append(i)
        for s in range(2):
            reads.setdefault(("w", c), []).append((4 * c + 2 * s, c % NW))
            reads.setdefault(("h", 2 * c + s), []).append((4 * c + 2 * s, (2 * c + s) % NH))
        for j in issued[:len(issued) - (NW - 2)]:
            landed.setdefault(("w", j), 4 * c + 3)
    slots0 = 4 * nch + 1
    # G = 1
    issued = list(range(NH))
    fills[("h", NH - 1)] = (0, (NH - 1) % NH)
    for i in range(NH - 1):
        landed[("h", i)] = -1
    for c in range(nch):
        for s in range(2):
            q = 2 * c + s
            reads[("w", c)].append((2 * q + 1, c % NW))
            reads[("h", q)].append((2 * q + 1, q % NH))
            for j in issued[:len(issued) - (NH - 2)]:
                landed.setdefault(("h", j), 2 * q + 1)
            i = q + NH
            fills[("h", i)] = (2 * q + 2, i % NH)
            issued.append(i)
    slots1 = 4 * nch + 1
    assert slots0 == slots1
    for (op, i), rs in reads.items():
        for slot, stage in rs:
            assert landed[(op, i)] < slot  # waited for in an earlier slot
            for (fop, j), (fs, fst) in fills.items():
                if fop == op and j > i and fst == stage:
                    assert fs > slot  # the next fill of the stage is requested in a later slot


@pytest.mark.parametrize("rb", SHAPES)
@pytest.mark.parametrize("R,V", [(129, 13057), (155, 300), (520, 4099), (576, 257), (2048, 2500)])
def test_untruncated_dense_row_accesses_stay_in_bounds(R, V, rb):
    """The untruncated epilogue's 16-byte accesses to the dense rows [R][tiles * 256]: parked
    expert logits and y stored where the row exists, loads from rows clamped to the last one."""
    g = _geo(rb)
    zstride = (V + TT - 1) // TT * TT
    b, vb, lane = np.meshgrid(np.arange(rb), np.arange(4), LANE, indexing="ij")
    stored = np.zeros((R, zstride // 4), np.int32)
    for tile, row0 in _tiles(R, V, g["TR"]):
        for wave in range(8):
            wt, G = wave % 4, wave // 4
            row = row0 + G * 16 * rb + 16 * b + lane % 16
            col = tile * TT + 64 * wt + 4 * (lane // 16) + 16 * vb
            assert np.all(col % 4 == 0) and np.all(col + 4 <= zstride)
            load = np.minimum(row, R - 1).astype(np.int64) * zstride + col
            assert np.all(load >= 0) and np.all(load + 4 <= R * zstride)
            ok = row < R
            np.add.at(stored, (row[ok], col[ok] // 4), 1)
    assert np.all(stored == 1)  # every 16 bytes of every row by one lane
