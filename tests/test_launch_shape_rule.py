"""The launch-shape rule on the CPU: a shape that gives the shots per block
alone is answered the same way at every batch size."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2609_38139_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("shapes") / "shapes")
    subprocess.run([HIPCC, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                    os.path.join(HERE, "launch_shape", "shapes.cpp"), "-o", exe, "-L", PKG, "-llaim",
                    f"-Wl,-rpath,{PKG}"], check=True)

    def run(lines):
        r = subprocess.run([exe], input="\n".join(" ".join(map(str, x)) for x in lines) + "\n", capture_output=True,
                           text=True, check=True)
        return [[int(v) for v in row.split()] for row in r.stdout.strip().split("\n")]
    return run


# (check degree, qubit degree, regular, on the 2D toric lattice, qubits per check)
FAMILIES = [(2, 2, 1, 0, 1), (4, 2, 1, 0, 2), (4, 2, 1, 1, 2), (6, 2, 1, 0, 3), (4, 4, 1, 0, 1), (6, 3, 1, 0, 2),
            (6, 2, 0, 0, 3), (8, 4, 0, 0, 2)]
CHECKS = (16, 36, 64, 72, 100, 125, 128, 169, 216, 256, 257, 288, 432, 441, 448, 512, 513, 576, 640, 648, 784, 900,
          1000, 1024)


def test_a_shape_with_shots_per_block_alone_is_accepted_at_every_batch_size(shapes):
    rows = []
    for dc, dv, regular, lattice, per in FAMILIES:
        for m in CHECKS:
            if lattice and m % 16:
                continue
            for bp in (0, 1):
                for seq in (0, 1):
                    for spb in (1, 2, 3, 4, 5, 8, 13, 16, 31, 40):
                        rows.append((m, m * per, dc, dv, regular, lattice, bp, seq, spb))
    got = shapes(rows)
    assert len(got) == len(rows)
    accepted = 0
    for row, out in zip(rows, got):
        m, spb = row[0], min(row[8], 31)
        full, per_batch = out[0], [out[1 + 4 * i:5 + 4 * i] for i in range((len(out) - 1) // 4)]
        oks = {p[0] for p in per_batch}
        assert len(oks) == 1, (row, out)  # the answer does not depend on the batch
        if full:  # and is yes wherever the block written out in full runs
            assert oks == {1}, (row, out)
        for ok, nt, cpt, lanes in per_batch:
            if ok:
                accepted += 1
                assert nt * spb <= 1024 and nt // lanes * cpt >= m, (row, out)
    assert accepted > 10000
