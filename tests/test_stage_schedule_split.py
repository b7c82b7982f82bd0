"""CPU model of the fused stage kernel's LDS bookkeeping in its three barrier schedules (host
logic, no GPU).

Per step `it` (entering plane L = it - 2R, gradient plane a = L - R, output plane o = a - R):
  - the point fields and u of a go to one of NP buffers before the first barrier;
  - after it, every column forms its gradient at a from that buffer and stores the x/y nested
    pairs (NW buffers) and the z pair (own column);
  - the x and y sums run on plane a after a second barrier (schedule 0), or on plane a - 1 after
    the first (schedules 1 and 2), and read the point fields and the nested pairs of that plane;
  - their result waits in registers (0, 1: the same thread adds the z sums) or in one of R LDS
    buffers (2: another wavefront adds them, from the next barrier on).
The model replays the steps and checks that every read finds the plane it expects, written
before a barrier that precedes the read, and that nothing is written and read by different
threads between the same two barriers.
"""
import itertools

import pytest


def replay(R, zc, DB, NP=None, NW=None, npart=None):
    NP = (3 if DB else 2) if NP is None else NP
    NW = (2 if DB else 1) if NW is None else NW
    npart = R if npart is None else npart
    lag = 1 if DB else 0
    slots, access, phase = {}, {}, 0

    def write(arr, slot, plane):
        slots[(arr, slot)] = (plane, phase)
        access.setdefault((arr, slot, phase), set()).add("w")

    def read(arr, slot, plane):
        got, ph = slots[(arr, slot)]
        assert got == plane, (arr, slot, got, plane)
        assert ph < phase, (arr, slot, plane, "read in the phase it was written")
        access.setdefault((arr, slot, phase), set()).add("r")

    waiting, outputs = {}, []
    for it in range(zc + 4 * R):
        L = it - 2 * R
        a, o = L - R, L - 2 * R
        do_grad, do_out = it >= 2 * R, it >= 4 * R
        if do_grad:
            write("plane", it % NP, a)
        phase += 1
        if do_grad:
            read("plane", it % NP, a)
            write("pairs", it % NW, a)
        if DB == 0:
            phase += 1
        if 3 * R + lag <= it < zc + 3 * R + lag:
            b = a - lag
            read("plane", (it - lag) % NP, b)
            read("pairs", (it - lag) % NW, b)
            if DB == 2:
                write("part", it % npart, b)
            else:
                waiting[b] = True
        if do_out:
            if DB == 2:
                read("part", (it + 1) % npart, o)
            else:
                assert waiting.pop(o)
            outputs.append(o)
    races = [k for k, v in access.items() if len(v) > 1]
    assert not races, races[:4]
    assert outputs == list(range(zc))


@pytest.mark.parametrize("R,zc,DB", [c for c in itertools.product((1, 2, 3, 4), (1, 2, 5, 11, 64), (0, 1, 2))
                                     if not (c[0] == 1 and c[2] == 2)])
def test_lds_schedules(R, zc, DB):
    replay(R, zc, DB)


@pytest.mark.parametrize("kw", [dict(DB=0, NP=1), dict(DB=1, NP=2), dict(DB=1, NW=1), dict(DB=2, NP=2),
                                dict(DB=2, NW=1), dict(DB=2, npart=1)])
def test_model_catches_one_buffer_too_few(kw):
    with pytest.raises(AssertionError):
        replay(2, 16, **kw)


def test_split_schedule_needs_a_radius_of_two():
    # at R = 1 the output plane's partial sums would be read in the step that forms them
    with pytest.raises((AssertionError, KeyError)):
        replay(1, 16, DB=2)


@pytest.mark.parametrize("total", list(range(1, 40)) + [961, 1024, 1089])
def test_workgroups_map_one_to_one_onto_xcd_runs(total):
    # workgroup w runs on XCD w % 8 and takes a consecutive share of the logical ids
    per, extra = total // 8, total % 8
    lam = [w % 8 * per + min(w % 8, extra) + w // 8 for w in range(total)]
    assert sorted(lam) == list(range(total))
    for k in range(8):
        run = lam[k::8]
        assert run == list(range(run[0], run[0] + len(run))) if run else True


@pytest.mark.parametrize("tiles_x,tiles_y", [(1, 1), (5, 3), (3, 4), (7, 9), (32, 32), (2, 13)])
def test_strip_order_visits_every_tile_once(tiles_x, tiles_y, rows_max=4):
    seen = set()
    for tile in range(tiles_x * tiles_y):
        strip, r = divmod(tile, rows_max * tiles_x)
        rows = min(rows_max, tiles_y - strip * rows_max)
        seen.add((r // rows, strip * rows_max + r % rows))
    assert seen == {(x, y) for x in range(tiles_x) for y in range(tiles_y)}
