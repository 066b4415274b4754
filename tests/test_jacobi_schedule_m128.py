"""The pair schedule of the M = 128 Jacobi sweep on its 512 threads: 64 pair
slots of 8 lanes, eight slots a wavefront, two steps to a pass.  After a pass's
even step k the slots q and q ^ 1 exchange partners by a lane swap; the odd step
writes its partner to LDS and the next pass loads its own, behind a workgroup
barrier only where (k + 2) is a multiple of eight.  Brute force over every
group, pass and slot, with which wavefront wrote each column last."""

M, NT = 128, 512
TPP, PSW = 8, 8


def _lower(q, h):
    return ((q >> h) << (h + 1)) | (q & ((1 << h) - 1))


def test_swapped_partners_written_columns_and_barriers():
    assert M // 2 * TPP == NT and 64 // TPP == PSW
    seen, barriers = set(), 1                           # the first group ends with one
    wave = lambda q: q * TPP // 64
    for q in range(M // 2):
        seen.add((2 * q, 2 * q + 1))
    for h in range(1, 7):
        low, kend = 1 << h, 2 << h
        fresh = {}                                      # column -> wavefront that wrote it, no barrier since
        for k in range(low, kend, 2):
            loaded = {q: _lower(q, h) ^ k for q in range(M // 2)}
            assert len(set(loaded.values())) == M // 2
            for q, j in loaded.items():
                assert (j >> h) & 1 and fresh.get(j, wave(q)) == wave(q), (h, k, q)
                seen.add((_lower(q, h), j))
            for q in range(M // 2):                     # the odd step: the neighbour's partner, by the swap
                j = _lower(q, h) ^ (k + 1)
                assert loaded[q ^ 1] == j and wave(q) == wave(q ^ 1)
                seen.add((_lower(q, h), j))
            fresh = {_lower(q, h) ^ (k + 1): wave(q) for q in range(M // 2)}
            if k + 2 < kend and (k + 2) % PSW == 0:
                barriers, fresh = barriers + 1, {}
        barriers += 1                                   # after the group
    assert len(seen) == M * (M - 1) // 2
    # inside a group: none up to h = 3, then one behind every eighth step but the last
    assert barriers == 7 + 0 + 1 + 3 + 7


def test_width_change_by_64_columns_overwrites_nothing_unread():
    """Doubles at stride 136 narrowed in place to floats at stride 136 by
    chunks of 16 values a thread, upwards, and widened back downwards."""
    LDB, LDF, CC = M + 8, M + TPP, 16 * NT // M
    assert CC == 64
    dbl = lambda c: (8 * c * LDB, 8 * c * LDB + 8 * M)
    flt = lambda c: (4 * c * LDF, 4 * c * LDF + 4 * M)
    overlap = lambda a, b: a[0] < b[1] and b[0] < a[1]
    for c in range(CC):                                 # the first chunk's floats, the second's doubles
        assert not any(overlap(flt(c), dbl(c2)) for c2 in range(CC, M))
    for c in range(CC, M):                              # downwards: the second chunk's doubles, the first's floats
        assert not any(overlap(dbl(c), flt(c2)) for c2 in range(CC))
    assert flt(M - 1)[1] <= 8 * M * LDB
