"""Host check of the exchange chains of the transforms split over grids of
128-thread workgroups (csrc/split_impl.h, ntt_split.hip, ks_split.hip), in the
mappings that the kernels have: forward grid A (7 -> 4 of a 1024-point index),
grid B (from n-9 down to 0, words stored at 6), inverse grid C (words loaded at
6, from 0 up to n-9) and grid D (4 -> 7), and key switching's middle grid, which
goes from grid B's end at 0 straight to grid C's start at 0.  Each exchange
starts where the one before ended, so a thread overwrites only entries that it
read itself; the exchanges of grids B and C stay inside a wave; those of A and D
are cross-wave and take the barrier.  With wave-local exchanges only, a kernel
that uses LDS otherwise orders that itself: key switching's middle grid has a
barrier between the digits' last stores and the other groups' reads and one
between those reads and the inverse's first exchange; the client's kernel runs
forward and inverse back to back, 0 -> 6 and then 6 -> 0; the rotation kernels
that stage a row in LDS have a barrier after the gather."""
import pytest

THREADS, E, BLOCK = 128, 8, 1024


def elem(lo, t, k):
    return (t & ((1 << lo) - 1)) | (k << lo) | ((t >> lo) << (lo + 3))


def fwd_b(logn):
    """Mappings of grid B's passes (split_b_rest)."""
    nb = logn - 6
    return [nb - 3 * (p + 1) for p in range(nb // 3)] + ([0] if nb % 3 else [])


def inv_c(logn):
    """Mappings of grid C's passes (inv_split_c_rest)."""
    nb = logn - 6
    rem = nb % 3
    return ([0] if rem else []) + [rem + 3 * p for p in range(nb // 3)]


def exchanges(mappings):
    """(from, to) of the exchanges between passes; equal mappings need none."""
    return [(a, b) for a, b in zip(mappings, mappings[1:]) if a != b]


def wave_sets(lo):
    return [{elem(lo, t, k) for t in range(64 * w, 64 * w + 64) for k in range(E)} for w in range(THREADS // 64)]


def check(seq):
    for (_, to), (frm, _) in zip(seq, seq[1:]):
        assert to == frm
    for frm, to in seq:
        for lo in (frm, to):
            assert sorted(elem(lo, t, k) for t in range(THREADS) for k in range(E)) == list(range(BLOCK))
        if frm <= 6 and to <= 6:
            assert wave_sets(frm) == wave_sets(to)
        else:
            assert wave_sets(frm) != wave_sets(to)


@pytest.mark.parametrize("logn", [12, 13, 14])
def test_grids_b_and_c_stay_inside_a_wave(logn):
    b, c = fwd_b(logn), inv_c(logn)
    assert b[-1] == 0 and c[0] == 0 and c[-1] == logn - 9 and b[0] == logn - 9
    for mappings in (b + [6], [6] + c, b + c):  # forward, inverse, key switching's middle grid
        seq = exchanges(mappings)
        check(seq)
        assert all(frm <= 6 and to <= 6 for frm, to in seq)
    for lo in b + c:  # every mapping addresses its own block of 512 elements a wave
        assert wave_sets(lo) == [set(range(512 * w, 512 * w + 512)) for w in range(2)]


def test_grids_a_and_d_are_cross_wave():
    for seq in ([(7, 4)], [(4, 7)]):
        check(seq)
        assert all(max(frm, to) > 6 for frm, to in seq)
    # the residue mapping: element v = tid + 128 k of grid A is residue v & 15, row v >> 4,
    # and key switching's grid D reads its partner's centred residues at the same place
    assert [elem(7, t, k) for t in (0, 5, 127) for k in (0, 7)] == [t + 128 * k for t in (0, 5, 127) for k in (0, 7)]


def test_forward_then_inverse_of_one_workgroup():
    """The client's kernel: the inverse's first exchange starts where the
    forward's last one ended."""
    for logn, loge in ((10, 3), (11, 3), (12, 3), (13, 3), (14, 4)):
        full, rem = logn // loge, logn % loge
        fwd = [logn - loge * (p + 1) for p in range(full)] + ([0] if rem else []) + [6]
        inv = [6] + ([0] if rem else []) + [rem + loge * p for p in range(full)]
        seq = exchanges(fwd) + exchanges(inv)
        for (_, to), (frm, _) in zip(seq, seq[1:]):
            assert to == frm
