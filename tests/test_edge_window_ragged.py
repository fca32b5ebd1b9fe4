"""The column arithmetic of the kernels' loads and stores for rows of any even
length that start anywhere, checked exhaustively on the CPU against a model of
the memory accesses. A lane loads E elements at `base` (its own column, or at an
edge the smallest mirrored column rounded down to a multiple of E) and at
base + E, and selects its elements from the two. Vectors go by 32-bit words and
may reach past the row: the words beyond the buffer resource read as 0. A row
of 2-byte elements may start at the upper half of a word; its resource then
starts at that word and a load takes one word more and shifts. Whatever a lane
selects has to be the element it stands for, and no access may touch a word
that holds nothing of the row; a store may touch nothing but the row."""
import pytest

from test_edge_window import mirror

FAR = 1 << 40          # the offset of an access that is dropped


def _words(n, size, odd):
    """The row's words as its resource shows them: per word its elements (2-byte:
    low and high half; None: nothing of the row), from the word it starts in."""
    if size == 4:
        return [[e] for e in range(n)]
    at = list(range(n))
    halves = ([None] if odd else []) + at
    halves += [None] * (len(halves) % 2)
    return [halves[i:i + 2] for i in range(0, len(halves), 2)]


def _load(words, x, E, size, odd):
    """E elements at column x, and the words touched."""
    if x == FAR:
        return [0] * E, []
    if size == 4:
        touched = range(x, x + E)
        flat = [words[w][0] if w < len(words) else 0 for w in touched]
        return flat, [w for w in touched if w < len(words)]
    count = max(1, E // 2) + (1 if odd and E > 1 else 0)
    first = 2 * x // 4
    halves = []
    touched = []
    for w in range(first, first + count):
        if w < len(words):
            touched.append(w)
            halves += words[w]
        else:
            halves += [0, 0]
    if E > 1:
        assert 2 * x % 4 == 0                      # vectors start at even columns
    skip = (x % 2 if E == 1 else 0) + (1 if odd and E > 1 else 0)
    return halves[skip:skip + E], touched


def _lanes(m_of, n, E, size, odd, starts):
    words = _words(n, size, odd)
    for x0 in starts:
        m = m_of(x0)
        plain = x0 >= 0 and x0 + E <= n
        base = x0 if plain else (min(m) & ~(E - 1))
        a, ta = _load(words, base, E, size, odd)
        b, tb = _load(words, FAR if plain else base + E, E, size, odd)
        sel = list(range(E)) if plain else [v - base for v in m]
        assert all(0 <= s < 2 * E for s in sel)
        assert [(a + b)[s] for s in sel] == m, (n, E, size, odd, x0)
        for w in ta + tb:
            assert any(e is not None for e in words[w])


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("size,E", [(4, 2), (4, 4), (4, 8), (2, 2), (2, 4), (2, 8)])
def test_forward_columns(size, E, odd):
    if size == 4 and odd:
        odd = False                                # 4-byte rows start at words
    for n in range(2, 84, 2):
        _lanes(lambda x0: [mirror(x0 + k, n) for k in range(E)], n, E, size, odd,
               range(-4 * E, n + 4 * E, E))


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("size,E", [(4, 2), (4, 4), (2, 2), (2, 4)])
def test_inverse_phase_columns(size, E, odd):
    if size == 4 and odd:
        odd = False
    for nq in range(1, 60):
        w = 2 * nq
        starts = range(-4 * E, nq + 4 * E, E)
        _lanes(lambda q: [mirror(2 * (q + i), w) >> 1 for i in range(E)], nq, E, size, odd, starts)
        _lanes(lambda q: [(mirror(2 * (q + i) + 1, w) - 1) >> 1 for i in range(E)], nq, E, size,
               odd, starts)


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("N", [2, 4, 8])
def test_stores_of_two_byte_rows(N, odd):
    """Every element of the row is written once, by its own lane, and nothing
    else is: whole vectors (at odd rows a half, whole words, a half) inside the
    row, one half at a time in the row's last lane."""
    for n in range(1, 70):
        written = {}
        shift = 1 if odd else 0
        for x0 in range(0, n + 2 * N, N):
            if x0 >= n:
                continue                           # the lane does not store
            if x0 + N <= n:
                halves = list(range(x0 + shift, x0 + shift + N))
                if odd:                            # a half, words, a half
                    assert halves[0] % 2 == 1 and halves[-1] % 2 == 0
                    assert all(h % 2 == 0 for h in halves[1:-1:2])
                else:
                    assert halves[0] % 2 == 0
            else:
                halves = [x0 + shift + i for i in range(N) if x0 + i < n]
            for i, h in enumerate(halves):
                assert h not in written
                written[h] = x0 + i
        assert written == {e + shift: e for e in range(n)}
