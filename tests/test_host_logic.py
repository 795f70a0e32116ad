"""CPU-only checks of rules that the kernels rely on, written out again in Python from
their descriptions (the device code is not run here): an item of the persistent FFN kernels stays on one XCD as far
as contiguous ranges let it (tests/test_tile_units.py walks the numbering itself), and the cut of a long
expert into equal work items must give positive, tile-sized items that add up to the expert's rows."""
import glob
import os
import random
import re


def units_of(group: int, total: int, groups: int = 256, xcds: int = 8):
    """Workgroups go to the XCDs round-robin; each XCD has a contiguous range of the units, which its workgroups take in
    turn."""
    x, q, r = group % xcds, total // xcds, total % xcds
    first = x * q + min(x, r)
    return list(range(first + group // xcds, first + q + (1 if x < r else 0), groups // xcds))


def test_every_unit_has_one_workgroup_and_an_item_stays_on_one_xcd():
    rng = random.Random(7)
    for _ in range(300):
        items, parts = rng.randint(1, 700), rng.choice([1, 2, 3, 6, 8, 11, 12, 16, 24])
        total = items * parts
        owner, seen = {}, []
        for g in range(256):
            units = units_of(g, total)
            seen += units
            for u in units:
                owner.setdefault(u // parts, set()).add(g % 8)
        assert sorted(seen) == list(range(total))
        # an item's parts meet on one XCD except where an XCD's range ends inside an item (at most 7 items in all)
        assert sum(1 for xs in owner.values() if len(xs) > 1) <= 7, (items, parts)


def cut_expert(rows: int, item_rows: int):
    """Items of one expert: as many as rows / item_rows rounded up; from 128-row items on, two to
    four items share the rows equally, rounded up to 16-row tiles."""
    n = -(-rows // item_rows)
    per = item_rows
    if item_rows >= 128 and 2 <= n <= 4:
        per = (-(-rows // n) + 15) // 16 * 16
    return [min(per, rows - j * per) for j in range(n)]


def test_long_experts_are_cut_into_positive_tile_sized_items():
    for item_rows in (32, 64, 96, 128, 160, 192, 256):
        for rows in range(1, 4 * item_rows + 40):
            items = cut_expert(rows, item_rows)
            assert sum(items) == rows
            assert all(0 < c <= item_rows for c in items), (rows, item_rows, items)
            assert all(c % 16 == 0 for c in items[:-1]) or item_rows < 128 or len(items) > 4


def test_inline_assembly_declares_the_registers_it_writes():
    """An asm statement that writes m0 has to say so: the compiler may keep a value of its own there."""
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_07616_amd", "csrc")
    found = 0
    for path in glob.glob(os.path.join(csrc, "*.h*")):
        for text in re.findall(r"asm volatile\((.*?)\);", open(path).read(), re.S):
            if re.search(r"\bs_mov_b32 m0\b", text):
                found += 1
                assert '"m0"' in text.rsplit(":", 1)[1], (path, text)
    assert found == 2
