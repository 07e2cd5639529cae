"""The benchmark's count of the orbital operator's stored rows (no GPU): the pairs
of extended nodes on one line of a cell, counted one by one on small meshes."""
import pytest

from synth import small_workload


@pytest.mark.parametrize("name", ["tiny_q1", "tiny_q2", "tiny_q3"])
def test_orbital_row_entries(name):
    import bench
    import paper_2301_02387_amd as mh
    mesh = mh.Mesh.from_workload(small_workload(name))
    P, NE = mesh.info["p"] + 1, mesh.info["n_dof"] + mesh.info["n_hang"]
    pairs = set()
    for cell in mesh.cells()[0]:
        for t, i in enumerate(cell):
            a, b, c = t % P, (t // P) % P, t // (P * P)
            for q in range(P):
                for j in (cell[(c * P + b) * P + q], cell[(c * P + q) * P + a], cell[(q * P + b) * P + a]):
                    if i < NE and j < NE:
                        pairs.add((int(i), int(j)))
    entries = bench.orbital_row_entries(mesh)
    assert entries == len(pairs)
    assert bench.orbital_row_bytes(entries, NE) == 4 * (NE + 1) + 12 * entries
    assert bench.orbital_row_bytes(entries, NE, 1, True, True) == 4 * (NE + 1) + 36 * entries
