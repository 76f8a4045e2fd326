"""Work lists of batches of boards: every tile plane stepped once, none in pieces below
two planes where a tile is cut, and the device shared evenly.

The planning is host code, run without a GPU (tests/host/host_logic.cpp, `plan`).
"""
import pytest

from test_host_cpu import _check_cover, _parse_plan, _tiles, host_logic  # noqa: F401

TY, ROWS, SLOTS = 14, 11, 32   # 64 x 14 x 2 on 256 compute units: 32 blocks per XCD

CASES = {
    # boards (nx, ny, nz)
    "one_plane_boards": [(70, 20, 1)] * 3 + [(70, 20, 2)] * 2,
    "depths_21_to_91": [(48, 43, 21 + 5 * q) for q in range(15)],        # fewer tiles than blocks
    "deep_first": [(48, 43, 91 - 5 * q) for q in range(15)],
    "one_deep": [(48, 43, 20)] * 9 + [(48, 43, 400)],
    "as_many_tiles_as_blocks": [(48, 43, 30)] * 64,
    "one_tile_more": [(48, 43, 30)] * 64 + [(48, 11, 30)],
    "two_rounds_uneven": [(300, 200, 20 + q) for q in range(6)],
}


@pytest.mark.parametrize("name", list(CASES))
def test_batch_work_lists_cover_and_share(host_logic, tmp_path, name):  # noqa: F811
    boards = CASES[name]
    (tmp_path / "spec.txt").write_text("".join(f"{x} {y} {z} 2 0 0 -\n" for x, y, z in boards))
    order, spans, _, _ = _parse_plan(host_logic("plan", 64, TY, 2, 8 * SLOTS, tmp_path / "spec.txt"))
    assert len(spans) == 1 and len(spans[0]["lists"]) == 1
    ents = spans[0]["lists"][0][1]
    assert len(ents) % 8 == 0
    seen = {}
    for b, ix, iy, kb, ke in ents:
        if b >= 0:
            assert kb < ke
            seen.setdefault(order[b], []).append((ix, iy, kb, ke))
    assert set(seen) == set(range(len(boards)))
    for h, es in seen.items():
        nx, ny, nz = boards[h]
        _check_cover(es, _tiles(nx, ny, nz, 64, ROWS), nz, (name, h))
        whole = {}
        for ix, iy, kb, ke in es:
            whole.setdefault((ix, iy), []).append(ke - kb)
        assert all(len(v) == 1 or min(v) >= 2 for v in whole.values())
        assert all(len(v) <= 16 for v in whole.values())
    # planes that the device walks in sequence, a block's own start (4 planes' worth)
    # included: never more than uncut tiles would take, and within 20 % (plus a
    # tile's granularity of two planes) of an even share where no tile is deeper
    tiles = [(h, nz) for h, (nx, ny, nz) in enumerate(boards) for _ in _tiles(nx, ny, nz, 64, ROWS)]
    run = len(ents) // 8
    walk = 0
    for x in range(8):
        real = [ke - kb + 4 for b, _, _, kb, ke in ents[x * run:(x + 1) * run] if b >= 0]
        slots = [0] * SLOTS
        for t in real:                       # blocks go to the first free slot, in order
            i = slots.index(min(slots))
            slots[i] += t
        walk = max(walk, max(slots))
    if len(tiles) <= 8 * SLOTS:
        assert walk <= max(nz for _, nz in tiles) + 4
        share = sum(nz for _, nz in tiles) / (8 * SLOTS)
        if name in ("depths_21_to_91", "deep_first"):
            assert walk - 4 <= 1.2 * share + 2
