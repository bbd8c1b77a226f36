"""The kernels' address arithmetic, restated on the host (CPU only).

The HIP kernels read spd through 32-bit buffer offsets and index per-lane
LDS tables and histograms by spd bytes. These tests restate each address
expression of the kernels (the constants are read from the sources) and
check the extremes the host validation admits: every spd offset stays below
the buffer range 2^31 - 1 at the largest row stride, every byte value
0..255 lands on a table/histogram entry inside its LDS object, and the
128-bucket layout's remap sends every byte >= 128 to the padding bucket."""
import re
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parents[1] / "paper_2609_34420_amd" / "csrc"
RANGE = 0x7FFFFFFF                     # num_records of the kernels' buffer resources


def _const(name, fname="api.hip"):
    text = (CSRC / fname).read_text()
    m = re.search(rf"constexpr int64_t {name} = \(1LL << (\d+)\) - (\d+);", text)
    return (1 << int(m.group(1))) - int(m.group(2))


K_MAX_LD = _const("kMaxLd")


def perm(s0, s1, sel):
    """v_perm_b32: byte i of the result is byte sel_i of (s0:s1), where
    selectors 0..3 pick s1's bytes, 4..7 s0's, and 0x0c gives 0."""
    b = [(s1 >> (8 * i)) & 0xFF for i in range(4)] + [(s0 >> (8 * i)) & 0xFF for i in range(4)]
    out = 0
    for i in range(4):
        s = (sel >> (8 * i)) & 0xFF
        out |= (0 if s == 0x0C else b[s]) << (8 * i)
    return out


def test_max_stride_constant_matches_the_header():
    text = (Path(__file__).resolve().parents[1] / "include" / "gt_attn.h").read_text()
    assert "2^25 - 16" in text and K_MAX_LD == 2 ** 25 - 16


@pytest.mark.parametrize("ld", [K_MAX_LD, K_MAX_LD - 16, 131072, 64])
def test_query_stationary_spd_offsets(ld):
    """Forward and dQ: a wave's resource starts at its first query row; lane
    offset (row - first) ld + 16 g, key offset jt + 32 kb as the scalar part;
    a 16-byte load. Forward waves own 64 rows, dQ waves 32."""
    Sk = ld                              # the widest key block the stride admits
    for rows in (64, 32):
        v = (rows - 1) * ld + 16          # largest lane offset (g = 1)
        s = (Sk - 64) + 32                # last tile, second 32-key block
        assert v + s + 15 <= RANGE, (ld, rows)


@pytest.mark.parametrize("ld", [K_MAX_LD, 131072, 4096])
def test_key_stationary_spd_offsets(ld):
    """dK/dV: column gathers read bytes i_base + 16 g + r (r < 16) of the
    key's column from a resource at row i_base: lane offset 16 g ld + key,
    scalar offset r ld; the transposed rows (spd_t) are used only when
    256 ld < 2^31, lane offset (key - key0) ld + 16 g, scalar offset i_base
    <= ld - 16, one 16-byte load."""
    key = 255
    assert 16 * ld + key + 15 * ld <= RANGE
    if 256 * ld < 2 ** 31:
        assert (255 * ld + 16) + (ld - 16) + 15 <= RANGE


def test_forward_lane_table_addresses():
    """Forward and dQ: entry (b, lane) at byte 256 b + 4 lane of a 64 KiB
    per-lane table, from one permute: every byte value has an entry."""
    for lane in (0, 1, 31, 32, 63):
        for r in range(4):
            for b in (0, 1, 127, 128, 255):
                w = b << (8 * r)
                a = perm(w, lane * 4, 0x0C0C0000 | ((4 + r) << 8))
                assert a == 256 * b + 4 * lane
                assert 0 <= a and a + 4 <= 256 * 64 * 4


def _clamp128(b):
    return 0x7F if b & 0x80 else b


def test_key_stationary_table_and_histogram_128():
    """dK/dV with at most 127 buckets: 32 copies (lane & 31) of a 128-bucket
    layout at byte 64 KiB, 8-byte entries; the histogram entry 32 KiB past
    the table entry. Bytes >= 128 are first mapped to the padding bucket 127.
    Every (byte, lane) lands inside the table and histogram of its copy."""
    tab_base, ent = 1 << 16, 128 * 32
    seen = set()
    for lane in range(64):
        cpyb = (lane & 31) * 8 | tab_base
        for b in range(256):
            bc = _clamp128(b)
            assert bc < 128 and (bc == b or bc == 127)
            a = perm(bc, cpyb, 0x0C020400)
            assert a == tab_base + 256 * bc + 8 * (lane & 31)
            idx = (a - tab_base) // 8
            assert 0 <= idx < ent and idx % 32 == (lane & 31)
            hist = a + ent * 8
            assert tab_base + ent * 8 <= hist < tab_base + 2 * ent * 8
            seen.add(idx)
    assert len(seen) == ent


def test_key_stationary_table_and_histogram_256():
    """Past 127 buckets where the tiles take the whole 64 KiB below the table
    (d = 64, four query groups): 16 copies (lane & 15) of a 256-bucket layout,
    entry address (b << 7) | copy offset | base."""
    tab_base, ent = 1 << 16, 256 * 16
    for lane in range(64):
        cpyb = (lane & 15) * 8 | tab_base
        for b in range(256):
            a = (b << 7) | cpyb
            idx = (a - tab_base) // 8
            assert 0 <= idx < ent and idx == b * 16 + (lane & 15)
            assert a + ent * 8 < tab_base + 2 * ent * 8


def test_key_stationary_table_and_histogram_256_halved():
    """Past 127 buckets elsewhere: 32 copies (lane & 31), the histogram from 64
    KiB at the permuted address, the 4-byte table from 32 KiB at half of it."""
    hist_base, tab_base, ent = 1 << 16, 1 << 15, 256 * 32
    seen = set()
    for lane in range(64):
        cpyb = (lane & 31) * 8 | hist_base
        for b in range(256):
            a = perm(b, cpyb, 0x0C020400)
            assert (a - hist_base) // 8 == b * 32 + (lane & 31) < ent
            t = a >> 1
            assert t % 4 == 0 and (t - tab_base) // 4 == b * 32 + (lane & 31)
            assert tab_base <= t < tab_base + ent * 4 <= hist_base
            seen.add(a)
    assert len(seen) == ent


def test_histogram_fixed_point_range():
    """Every histogram term is round(dS 2^F) with |dS| 2^F <= 2^30: a copy's
    64-bit sum of the 2 lanes x 8 waves x N queries that can share it stays
    below 2^63 for every N the stride limit admits."""
    terms = 2 * 8 * K_MAX_LD
    assert terms * 2 ** 30 < 2 ** 63


@pytest.mark.parametrize("Sk", [1, 3, 16, 17, 31, 64, 100, 127, 130])
@pytest.mark.parametrize("addr", [0, 1, 2, 3, 5, 14, 15])
def test_spd_groups_at_any_address(Sk, addr):
    """Forward, dQ and dK/dV: the group of 16 keys from key j of a buffer's
    last row, which starts at byte `addr` past a 16-byte boundary and ends the
    buffer. The resource starts at the boundary and ends with the dword of the
    last key; dwords past its end read 0. Rows on dword boundaries are loaded
    as 4 dwords; others as the 5 dwords from the address rounded down, shifted
    by the address mod 4. Every key's byte arrives in place, and no dword is
    read that holds no byte from the boundary on to the last key."""
    row = [(7 * j + 3) % 251 + 1 for j in range(Sk)]
    end4 = (addr + Sk + 3) & ~3                # num_records of the resource
    assert end4 - (addr + Sk) < 4
    buf = [0xEE] * addr + row + [0xEE] * (end4 - addr - Sk)

    def dwords(a, n):
        assert a % 4 == 0 and a >= 0
        return sum((buf[x:x + 4] if x + 4 <= end4 else [0] * 4 for x in range(a, a + 4 * n, 4)), [])

    for j in range(0, (Sk + 63) // 64 * 64, 16):
        a = addr + j
        w = dwords(a & ~3, 5)[a & 3:(a & 3) + 16]   # v_alignbyte over the 5 dwords
        n = max(0, min(16, Sk - j))
        assert w[:n] == row[j:j + n]
        if addr % 4 == 0:
            assert dwords(a, 4)[:n] == row[j:j + n]


def _raw_loads(text):
    """(function, scalar offset) of every raw buffer load in a source."""
    out = []
    for m in re.finditer(r"__builtin_amdgcn_raw_buffer_load_\w+\(", text):
        depth, i, args, start = 1, m.end(), [], m.end()
        while depth:
            c = text[i]
            if c in "([{":
                depth += 1
            elif c in ")]}":
                depth -= 1
            if (c == "," and depth == 1) or depth == 0:
                args.append(text[start:i].strip())
                start = i + 1
            i += 1
        fn = re.findall(r"__forceinline__ \S+ (\w+)\(", text[:m.start()])
        out.append((fn[-1] if fn else "", args[2]))
    return out


def test_loads_that_may_pass_the_end_have_no_scalar_offset():
    """A scalar offset is not part of a raw buffer load's range check (or is
    subtracted from the end, which then goes negative), so only loads that are
    inside whatever the lane have one: those of buf_u128_inside, taken by the
    query-stationary kernels on whole tiles, by the short forward on whole key
    blocks and by dK/dV with a transpose on whole key blocks."""
    callers = []
    for f in sorted(CSRC.iterdir()):
        if f.suffix not in (".hip", ".hpp"):
            continue
        text = f.read_text()
        for fn, soff in _raw_loads(text):
            assert soff in ("0", "0u") or fn == "buf_u128_inside", (f.name, fn, soff)
        for m in re.finditer(r"(if constexpr \([^\n]*?\)|else)\s*(//[^\n]*)?\n\s*buf_u128_inside\(", text):
            callers.append((f.name, m.group(1)))
        assert text.count("buf_u128_inside(") == (f.name == "common.hpp") + sum(c[0] == f.name for c in callers)
    assert callers == [("bwd_dkdv.hip", "if constexpr (!KTAIL)"), ("fwd_short.hip", "else"),
                       ("stage.hpp", "if constexpr (whole_keys(ROWS))")]
    text = (CSRC / "fwd_short.hip").read_text()
    assert re.search(r"else if constexpr \(TAIL\)\n\s*buf_u128\(.*\n\s*else\n\s*buf_u128_inside", text)


# (first row's address, rows of the wave from its first on, keys, row stride,
# tile, the groups' parts)
@pytest.mark.parametrize("Sk", [1, 5, 17, 33, 100, 200, 257])
@pytest.mark.parametrize("rows,pad,addr", [(1, 0, 0), (1, 0, 3), (2, 3, 5), (3, 4, 8), (64, 1, 13)])
@pytest.mark.parametrize("tile,parts", [(64, (0,)), (128, (0, 32, 64, 96)), (256, (0, 64, 128, 192))])
def test_query_stationary_spd_reads_stay_in_the_matrix(Sk, rows, pad, addr, tile, parts):
    """Forward and dQ: the load of a 16-key group whose first key may lie past
    the last one, or be none of the wave's rows. Its resource starts at the
    group's key (from the 16-byte boundary below the first row on) and ends
    with the dword of the last row's last key, empty past it; only the lane
    offset is compared with that end. No dword past the end is touched and the
    keys that exist arrive in place."""
    ld = Sk + pad
    rem = addr & 15
    end = (rem + (rows - 1) * ld + Sk + 3) & ~3          # from the boundary on
    for t in range((Sk + tile - 1) // tile):
        for part in parts:
            for kb in range(0, tile // len(parts), 32):
                skip = t * tile + part + kb
                records = max(0, end - skip)
                for row in {0, rows - 1}:
                    for g in (0, 1):
                        v = row * ld + 16 * g + rem
                        sh = v & 3
                        touched = [skip + v - sh + 4 * i for i in range(5) if v - sh + 4 * i + 4 <= records]
                        assert all(0 <= x and x + 4 <= end for x in touched)
                        got = {x + i for x in touched for i in range(4)}
                        first = skip + 16 * g
                        for j in range(first, min(first + 16, Sk)):
                            assert rem + row * ld + j in got


@pytest.mark.parametrize("N", list(range(1, 70)) + [96, 100, 130, 200, 224, 255, 256])
def test_short_spd_reads_stay_in_the_matrix(N):
    """Short forward (key block j of the lane's row, at least two blocks) and
    short backward (query block qb of every wave slot, also past the last
    block): as above, with the whole offset in the lane and with the block's
    rows in the resource's start."""
    lgp = 0 if N > 128 else (1 if N > 64 else (2 if N > 32 else 3))
    for rem in (0, 1, 4, 15):
        end = (rem + (N - 1) * N + N + 3) & ~3
        for j in range(0, 32 * max(2, (N + 31) // 32), 32):
            for row in (0, N // 2, N - 1):
                for g in (0, 1):
                    v = (row * N + 16 * g + rem & ~3) + j
                    touched = [v + 4 * i for i in range(5) if v + 4 * i + 4 <= end]
                    need = {rem + row * N + k for k in range(j + 16 * g, min(j + 16 * g + 16, N))}
                    assert need <= {x + i for x in touched for i in range(4)}
        for qb in range(8 >> lgp):
            skip = qb * 32 * N
            assert skip % 16 == 0
            records = max(0, end - skip)
            for lane in (0, 1, 31, 62, 63):
                for wl in range(8 >> lgp):
                    v = (lane >> 1) * N + 16 * (lane & 1) + wl * 32 + rem & ~3
                    touched = [skip + v + 4 * i for i in range(5) if v + 4 * i + 4 <= records]
                    assert all(x + 4 <= end for x in touched)
                    i = qb * 32 + (lane >> 1)
                    first = wl * 32 + 16 * (lane & 1)
                    if i < N:
                        need = {rem + i * N + k for k in range(first, min(first + 16, N))}
                        assert need <= {x + b for x in touched for b in range(4)}


@pytest.mark.parametrize("N", list(range(16, 700, 16)) + [1008, 1024, 1040, 4096, 4112])
def test_transposed_spd_reads_stay_in_the_matrix(N):
    """dK/dV with spd_t (N a multiple of 16): a whole key block's loads are
    inside the matrix by themselves (the resource ends with the block, but is
    not relied on); the partial block's are held by the lane offset."""
    for split, tile in ((1, 64), (2, 64), (2, 128), (4, 128)):
        bk, nsub = 256 // split, tile // (32 * split)
        last32, ntiles = (N - 1) & ~31, (N + tile - 1) // tile
        starts = {t * tile + qs * nsub * 32 + 32 * s for t in {0, ntiles - 1} for qs in range(split)
                  for s in range(nsub)}
        for key0 in {0, (N - 1) // bk * bk, max(0, (N // bk - 1) * bk)}:
            rows = min(bk, N - key0)
            for i in starts:
                if rows == bk:
                    soff = last32 if tile > bk and i > last32 else i
                    assert key0 * N + (bk - 1) * N + 16 + soff + 16 <= N * N
                    assert soff == i or i >= N         # the queries that exist are read in place
                else:
                    for row in {0, rows - 1}:
                        for g in (0, 1):
                            v = row * N + 16 * g + i
                            assert all(key0 * N + x + 4 <= N * N for x in range(v, v + 16, 4) if x + 4 <= rows * N)
