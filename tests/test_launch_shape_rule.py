"""The launch-shape rule on the CPU: which shapes it accepts, and the lines where
its choice changes."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2609_38139_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def build(tmp, name):
    exe = str(tmp / name)
    subprocess.run([HIPCC, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                    os.path.join(HERE, "launch_shape", name + ".cpp"), "-o", exe, "-L", PKG, "-llaim",
                    f"-Wl,-rpath,{PKG}"], check=True)

    def run(lines):
        r = subprocess.run([exe], input="\n".join(" ".join(map(str, x)) for x in lines) + "\n", capture_output=True,
                           text=True, check=True)
        return [[int(v) for v in row.split()] for row in r.stdout.strip().split("\n")]
    return run


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    return build(tmp_path_factory.mktemp("shapes"), "shapes")


@pytest.fixture(scope="module")
def wide(tmp_path_factory):
    return build(tmp_path_factory.mktemp("wide"), "wide")


# (check degree, qubit degree, regular, on the 2D toric lattice, qubits per check)
FAMILIES = [(2, 2, 1, 0, 1), (4, 2, 1, 0, 2), (4, 2, 1, 1, 2), (6, 2, 1, 0, 3), (4, 4, 1, 0, 1), (6, 3, 1, 0, 2),
            (6, 2, 0, 0, 3), (8, 4, 0, 0, 2)]
CHECKS = (16, 36, 64, 72, 100, 125, 128, 169, 216, 256, 257, 288, 432, 441, 448, 512, 513, 576, 640, 648, 784, 900,
          1000, 1024)


BATCHES = (0, 1, 40, 256, 1024, 4096, 65536, 2**31 - 1)


def test_a_shape_with_shots_per_block_alone_is_accepted_at_every_batch_size(shapes):
    rows = []
    for dc, dv, regular, lattice, per in FAMILIES:
        for m in CHECKS:
            if lattice and m % 16:
                continue
            for bp in (0, 1):
                for seq in (0, 1):
                    for spb in (1, 2, 3, 4, 5, 8, 13, 16, 31, 40):
                        rows += [(m, m * per, dc, dv, regular, lattice, bp, seq, spb, n, brief)
                                 for n in BATCHES for brief in (0, 1)]
    got = shapes(rows)
    assert len(got) == len(rows)
    accepted = 0
    for i in range(0, len(rows), 2 * len(BATCHES)):
        row, outs = rows[i], got[i:i + 2 * len(BATCHES)]
        oks = {o[1] for o in outs}
        assert len(oks) == 1, (row, outs)  # the answer depends neither on the batch nor on the rounds
        if outs[0][0]:  # and is yes wherever the block written out in full runs
            assert oks == {1}, (row, outs)
        for _, ok, nt, cpt, lanes, spb in outs:
            if ok:
                accepted += 1
                assert spb == min(row[8], 31) and nt * spb <= 1024 and nt // lanes * cpt >= row[0], (row, outs)
    assert accepted > 10000


def shape_of(shapes, m, dc, dv, regular, bp, nshots, per=2, brief=0):
    """(threads, checks per thread, lanes per check, shots per block) of the rule's own choice."""
    (_, ok, *shape), = shapes([(m, m * per, dc, dv, regular, 0, bp, 0, 0, nshots, brief)])
    assert ok
    return tuple(shape)


@pytest.mark.parametrize("nshots", [0, 8192, 65536])
def test_padded_degree_8_min_sum_never_takes_four_checks_per_thread(shapes, nshots):
    for m in (100, 200, 256, 257, 448, 600, 900, 1024):
        assert shape_of(shapes, m, 8, 4, 0, 0, nshots)[1] == (1 if m <= 256 else 2), m


@pytest.mark.parametrize("dc,dv,m,cpt", [
    (6, 3, 252, 1), (6, 3, 257, 2), (6, 3, 378, 2), (6, 3, 900, 2), (4, 4, 192, 1), (4, 4, 375, 2), (4, 4, 512, 2),
    (4, 4, 513, 1), (4, 4, 648, 1), (6, 2, 216, 4), (6, 2, 343, 2), (6, 2, 397, 4), (6, 2, 512, 4),
    (4, 2, 441, 8), (4, 2, 169, 4), (2, 2, 101, 4), (2, 2, 31, 1)])
def test_checks_per_thread_of_a_full_device_min_sum(shapes, dc, dv, m, cpt):
    assert shape_of(shapes, m, dc, dv, 1, 0, 0, per=1)[1] == cpt
    assert shape_of(shapes, m, dc, dv, 1, 0, 65536, per=1)[1] == cpt


@pytest.mark.parametrize("dc,dv,m,nshots,spb", [
    (2, 2, 9, 65536, 28), (2, 2, 15, 32768, 17), (2, 2, 31, 8192, 2), (2, 2, 31, 12000, 2), (2, 2, 31, 16384, 8), (2, 2, 31, 65536, 8),
    (2, 2, 64, 16384, 6), (2, 2, 64, 65536, 6), (2, 2, 101, 65536, 7), (4, 2, 25, 8192, 5), (4, 2, 25, 16384, 10),
    (4, 2, 25, 65536, 10), (4, 2, 121, 8192, 2), (4, 2, 121, 65536, 2), (6, 2, 64, 65536, 2), (6, 2, 125, 65536, 1),
    (6, 3, 72, 65536, 3), (6, 3, 36, 65536, 7), (4, 4, 81, 65536, 3), (4, 4, 192, 65536, 1), (2, 2, 9, 0, 28)])
def test_shots_per_block_of_small_codes(shapes, dc, dv, m, nshots, spb):
    assert shape_of(shapes, m, dc, dv, 1, 0, nshots, per=1)[3] == spb


@pytest.mark.parametrize("m,nshots,lanes", [(36, 65536, 2), (72, 65536, 2), (160, 65536, 2), (161, 65536, 1),
                                            (180, 32768, 1), (432, 32768, 1), (432, 0, 1), (432, 1024, 2),
                                            (432, 2048, 1), (450, 256, 2), (451, 256, 1), (72, 0, 2)])
def test_two_lanes_per_check_on_6_3_codes(shapes, m, nshots, lanes):
    assert shape_of(shapes, m, 6, 3, 1, 1, nshots)[2] == lanes


@pytest.mark.parametrize("m,nshots,lanes", [(256, 2048, 2), (257, 409, 2), (257, 410, 1), (324, 341, 2), (324, 342, 1),
                                            (324, 1, 2), (441, 1024, 1), (100, 4096, 2)])
def test_two_lanes_per_check_on_4_2_codes(shapes, m, nshots, lanes):
    assert shape_of(shapes, m, 4, 2, 1, 1, nshots)[2] == lanes


@pytest.mark.parametrize("dc,dv,m,nshots,cpt", [
    (6, 2, 216, 8192, 2), (6, 2, 216, 49152, 2), (6, 2, 216, 49153, 4), (6, 2, 343, 1 << 20, 2),
    (4, 4, 375, 5290, 1), (4, 4, 375, 5500, 2), (4, 4, 375, 1024, 1)])
def test_checks_per_thread_by_the_wavefronts_in_flight(shapes, dc, dv, m, nshots, cpt):
    assert shape_of(shapes, m, dc, dv, 1, 0, nshots, per=1)[1] == cpt


@pytest.mark.parametrize("dc,dv,m,bp,nshots,shape", [
    (4, 2, 64, 1, 2048, (128, 1, 2, 1)), (4, 2, 64, 1, 2049, (64, 1, 1, 1)), (4, 2, 64, 1, 8192, (64, 1, 1, 4)),
    (6, 3, 72, 1, 1024, (144, 1, 2, 1)), (6, 3, 72, 1, 1025, (72, 1, 1, 3)), (6, 3, 72, 1, 0, (72, 1, 1, 3)),
    (4, 2, 128, 1, 0, (128, 1, 1, 2)), (4, 2, 129, 1, 0, (65, 2, 1, 3)), (4, 2, 512, 1, 0, (256, 2, 1, 1)),
    (4, 2, 513, 1, 0, (129, 4, 1, 1)), (6, 3, 256, 1, 0, (256, 1, 1, 1)), (6, 3, 257, 1, 0, (129, 2, 1, 1)),
    (4, 4, 192, 1, 8192, (192, 1, 1, 1)), (4, 4, 648, 0, 5461, (648, 1, 1, 1)), (4, 4, 648, 0, 5462, (162, 4, 1, 1)),
    (4, 4, 512, 0, 0, (256, 2, 1, 1)), (6, 3, 900, 0, 4096, (450, 2, 1, 1)), (6, 3, 900, 0, 4097, (225, 4, 1, 1)),
    (4, 2, 81, 0, 7992, (41, 2, 1, 3)), (4, 2, 81, 0, 7993, (41, 2, 1, 6)), (6, 2, 125, 0, 8192, (63, 2, 1, 4)),
    (6, 2, 216, 0, 4096, (54, 4, 1, 1)), (6, 2, 216, 0, 8192, (54, 4, 1, 4)), (6, 2, 343, 0, 0, (86, 4, 1, 2)),
    (6, 2, 125, 0, 0, (63, 2, 1, 4)),
    (8, 4, 900, 0, 0, (450, 2, 1, 1))])
def test_decodes_of_at_most_two_rounds(shapes, dc, dv, m, bp, nshots, shape):
    assert shape_of(shapes, m, dc, dv, int(dc != 8), bp, nshots, per=1, brief=1) == shape


@pytest.mark.parametrize("m,nshots,cpt", [(320, 0, 1), (324, 0, 2), (324, 8192, 2), (324, 8022, 2), (324, 8021, 1),
                                          (484, 6016, 1), (400, 8192, 1), (512, 8192, 2), (513, 8192, 2),
                                          (576, 8192, 2), (576, 3527, 1), (576, 3528, 2), (1024, 8192, 2)])
def test_sum_product_checks_per_thread_on_4_2_codes(shapes, m, nshots, cpt):
    assert shape_of(shapes, m, 4, 2, 1, 1, nshots)[1:3] == (cpt, 1)


def test_wide_form_by_messages_and_shots(wide):
    rows = [((4900, 9800, 4, 2), 1, 1), ((22500, 45000, 4, 2), 1, 1), ((25600, 51200, 4, 2), 1, 0),
            ((32400, 64800, 4, 2), 1, 0), ((13824, 41472, 6, 2), 1, 1), ((17576, 52728, 6, 2), 1, 0),
            ((16384, 32768, 6, 3), 1, 1), ((25600, 51200, 6, 3), 1, 0), ((31944, 31944, 4, 4), 1, 1),
            ((4096, 8192, 4, 2), 0, 0), ((33000, 33000, 4, 4), 0, 0)]
    cases = [(code + (bp, n), few if n <= 128 else many)
             for code, few, many in rows for bp in (0, 1) for n in (1, 128, 129, 1024, 65536)]
    assert [r[0] for r in wide([c for c, _ in cases])] == [want for _, want in cases]
