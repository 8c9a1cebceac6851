"""How a call's paths and trees are cut into work items: host arithmetic,
compiled from the library's own headers and run here (CPU only)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CUS = 256


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """ask(commands): the check program's answers, one list of numbers each."""
    from paper_1705_03666_amd import build as B
    if shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("items") / "work_items_check")
    flags = [f for f in B.FLAGS if not f.startswith("--offload-arch")]
    obj = exe + ".o"
    subprocess.check_call([B._hipcc()] + flags + ["-c", os.path.join(HERE, "work_items_check.cpp"), "-o", obj])
    subprocess.check_call([B._hipcc(), obj, "-o", exe])

    def run(commands):
        r = subprocess.run([exe], input="\n".join(commands) + "\n", capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr
        out = [[int(v) for v in line.split()] for line in r.stdout.splitlines()]
        assert len(out) == len(commands)
        return out
    return run


def _items(trees, big, small):
    n_big = (trees - trees // 8) // big if trees > big and small < big else 0
    return n_big + -(-(trees - n_big * big) // small)


@pytest.mark.parametrize("trees", [1, 2, 63, 64, 65, 1000, 8191, 8193, 65537])
@pytest.mark.parametrize("big,small", [(1, 1), (7, 7), (64, 64), (256, 64), (1000, 256), (8192, 1024), (100000, 12500)])
def test_every_tree_is_in_one_item(ask, trees, big, small):
    for points in (1, 3):
        (n, _, _, ok), = ask([f"trees {points} {trees} {big} {small}"])
        assert ok == 1 and n == _items(trees, big, min(big, small))


def test_no_trees_no_items(ask):
    assert [a[0] for a in ask(["trees 5 0 8192 1024", f"bvp 5 0 8192 0 {CUS}", f"bvp 5 0 7 2 {CUS}"])] == [0, 0, 0]


@pytest.mark.parametrize("points,trees", [(1, 2**31 - 1), (2, 2**31 - 1), (2**24, 2**31 - 1), (2**30, 2**31 - 1),
                                          (1024, 10**8)])
def test_more_items_than_can_be_numbered(ask, points, trees):
    """Item sizes of a few trees: the search for a cut of at most 2^31 - 1
    items ends (it hung where only the large size grew), and the sizes still
    fit the 32 bits they are passed in."""
    for big, small in ((1, 1), (5, 5), (64, 8), (2**31 - 1, 1)):
        (n, b, s, _), = ask([f"trees {points} {trees} {big} {small}"])
        assert 0 < n * points <= 2**31 - 1
        assert 1 <= s <= b <= 2**31 and n == _items(trees, b, s)


def _partials(points, trees, times, chunk=8192, source=0, ask=None):
    (n, _, _, _), = ask([f"bvp {points} {trees} {chunk} {source} {CUS}"])
    return n * points * 48 * times


def test_boundary_partials_do_not_grow_with_the_trees(ask):
    """Branching with a boundary keeps 48 bytes per item and output time.
    Items of 8192 trees (the last eighth of 1024) needed 15 GB for 10^6 points
    x 10^5 trees x 11 times and 12 GB for 1024 x 10^8, which fits the card:
    no large call may need more than that, and the scratch of a call is
    bounded by its points and a fixed number of items a wavefront."""
    for points, trees in ((1024, 10**8), (10**6, 10**5), (1024, 10**5), (16, 2**31 - 1), (2**23, 1000), (1, 2**31 - 1),
                          (10**5, 10**6)):
        need = _partials(points, trees, 11, ask=ask)
        before = points * _items(trees, 8192, 1024) * 48 * 11
        assert need <= max(before, 256 << 20), (points, trees, need, before)
        # at most 32 large items a wavefront, half as many small ones, and a point's own remainders
        assert need <= (16 * CUS * 32 * 2 + 10 * points) * 48 * 11
    assert _partials(1024, 10**8, 11, ask=ask) < 300 << 20
    # the same from a schedule table that holds a small size
    assert _partials(1024, 10**8, 11, chunk=64, source=1, ask=ask) < 300 << 20


def test_boundary_item_sizes(ask):
    """An item size in the options is used as it is, as in the other entry
    points; one in the schedule table up to an eighth of a wavefront's share."""
    for chunk in (1, 7, 64, 100, 256, 700, 2048, 8192, 32768):
        small = max(min(256, chunk), chunk // 8)
        (n, _, _, ok), = ask([f"bvp 16 100000 {chunk} 2 {CUS}"])
        assert ok == 1 and n == _items(100000, chunk, min(small, chunk)), chunk
    # 1024 points x 10000 trees: 256 by default (share 312), the table's size where it is below that share
    big = [ask([f"bvp 1024 10000 {c} {f} {CUS}"])[0][1] for c, f in ((8192, 0), (128, 1), (300, 1), (8192, 1), (1, 2))]
    assert big == [256, 128, 300, 312, 1]
    # a small call: one tree per lane
    assert ask([f"bvp 5 3000 8192 0 {CUS}"])[0][1] == 64


def test_a_wavefront_per_node_stays_below_the_launch_limit(ask):
    """Calls take up to 2^30 nodes; a launch has fewer than 2^32 threads.  A
    wavefront each, until the launch takes its groups in turns."""
    sizes = [1, 4, 5, 4096, 65536, 65537, 2**26 - 1, 2**26, 2**30]
    for n, (threads,) in zip(sizes, ask([f"groups {n}" for n in sizes])):
        assert 0 < threads < 2**32 and threads % 256 == 0
        assert threads >= 64 * min(n, 65536)


def test_grids(ask):
    """A block for four items, as many as the chip holds of those asked for, at
    least one; up to the largest number of items."""
    for (per_cu, held, items), want in (((8, 5, 0), 1), ((8, 5, 1), 1), ((8, 5, 5), 2), ((8, 5, 10**6), 5 * CUS),
                                        ((2, 5, 10**6), 2 * CUS), ((8, 0, 10**6), 8 * CUS),
                                        ((4, 4, 2**31 - 1), 4 * CUS), ((4, 4, 2**31 - 3), 4 * CUS)):
        assert ask([f"grid {per_cu} {held} {items} {CUS}"]) == [[want]], (per_cu, held, items)
