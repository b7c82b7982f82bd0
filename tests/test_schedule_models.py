"""Models of bookkeeping that the GPU tests cannot see: the barriers of the marching residual step
(csrc/kernels_staged_march.h), the deal of an ensemble's workgroups to XCDs (fused_stage_kernel) and
the store offsets on long rows."""
import pytest


def _march(run, R, single):
    """Per role the list of (barriers passed, reads, writes), names with their buffer."""
    nb = 1 if single else 2
    cols, planes = [], []
    b = 0
    cols.append((b, [], []))                   # the window's first planes, own column only
    b += 1
    for j in range(run):
        b += 1                                 # the column's next plane has entered the window
        cols.append((b, ["part%d" % (j % nb)], []))
        if single and j + 1 < run:
            assert R >= 3                      # the barrier sits before the third neighbour pair
            b += 1                             # amid the z sums, after the partial sums were read
    ncols = b
    b = 0
    for it in range(run):
        planes.append((b, [], ["f%d" % (it % nb)]))
        b += 1
        planes.append((b, ["f%d" % (it % nb)], ["part%d" % (it % nb)]))
        if single:
            b += 1
    if not single:
        b += 1
    return cols, planes, ncols, b


@pytest.mark.parametrize("single", [False, True])
@pytest.mark.parametrize("run", [1, 2, 3, 7, 64])
def test_march_barriers(run, single):
    cols, planes, ncols, nplanes = _march(run, 6 if single else 3, single)
    assert ncols == nplanes                    # both roles pass every barrier
    writes = [(b, n, k) for k, (b, _, ws) in enumerate(planes) for n in ws if n.startswith("part")]
    reads = [(b, n, j) for j, (b, rs, _) in enumerate(cols) for n in rs]
    assert len(writes) == len(reads) == run
    for (wb, wn, _), (rb, rn, _) in zip(writes, reads):
        assert wn == rn and wb < rb            # plane j's sums: written a barrier before they are read
    for k, (rb, rn, _) in enumerate(reads):    # and not overwritten until a barrier after the read
        later = [wb for wb, wn, _ in writes[k + 1:] if wn == rn]
        assert all(wb > rb for wb in later)
    # a staged plane is read by all plane wavefronts after the barrier behind its writes, and written
    # again only a barrier after those reads
    f = [(b, "w", ws[0]) for b, _, ws in planes if ws[0].startswith("f")]
    r = [(b, "r", rs[0]) for b, rs, _ in planes if rs]
    for k, ((wb, _, wn), (rb, _, rn)) in enumerate(zip(f, r)):
        assert wn == rn and wb < rb
        assert all(b > rb for b, _, n in f[k + 1:] if n == rn)


def _lam(w, total, ninst, piece=16):
    xcd = w % 8
    dealt = total // (8 * piece) * (8 * piece) if ninst > 1 else 0
    per, extra, turn = (total - dealt) // 8, total % 8, w // 8
    if w < dealt:
        return (turn // piece * 8 + xcd) * piece + turn % piece
    return dealt + xcd * per + min(xcd, extra) + (turn - dealt // 8)


@pytest.mark.parametrize("ninst", [1, 2, 64])
def test_every_workgroup_is_dealt_once(ninst):
    for total in list(range(1, 420)) + [1023, 1024, 1025, 4095, 4099, 12345]:
        assert sorted(_lam(w, total, ninst) for w in range(total)) == list(range(total)), total


@pytest.mark.parametrize("size", [4, 8])
@pytest.mark.parametrize("ty", [4, 8, 16])
def test_store_offsets_stay_below_the_dropped_ones(size, ty):
    drop = bytes_ = 0x40000000
    edge = bytes_ // (ty * size)
    for nx in (16, 4096, edge - 1, edge, edge + 1, 2 ** 31 // 64):
        wide = ty * nx * size >= bytes_
        if not wide:
            assert ((ty - 1) * nx + nx - 1) * size + size <= drop
        else:
            assert nx >= edge                  # plain stores, every descriptor store dropped
