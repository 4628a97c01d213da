"""The 2D resident kernel loads as many columns per wavefront as its widest share has: whatever the
box, they lie inside the padded row (the kernel's own arithmetic, over every width it takes)."""
import pytest

WAVES = 16


@pytest.mark.parametrize("ny", [1, 64, 65, 128])
def test_loaded_columns_stay_in_the_row(ny):
    taken = 0
    for nx in range(3, 257):
        most, rows = -(-nx // WAVES), 1 if ny <= 64 else 2
        columns = 4 if most <= 4 else 8
        if most > 8 or columns * rows > 8:
            continue
        taken += 1
        pitch = -(-nx // 64) * 64
        first = [w * (nx // WAVES) + min(w, nx % WAVES) for w in range(WAVES + 1)]
        assert first[WAVES] == nx and all(b - a <= columns for a, b in zip(first, first[1:]))
        assert all(x + columns <= pitch for x in first[:WAVES])
    assert taken == (126 if ny <= 64 else 62)
