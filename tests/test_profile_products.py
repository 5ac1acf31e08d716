"""Which launches the traffic record counts as residue products, and which sources its
hash covers."""
import json

import pytest

from paper_2603_10634_amd import profile_summary as ps
from test_profile_summary import NS, _counters


def test_every_product_kernel_is_counted(tmp_path):
    copy = "__amd_rocclr_copyBuffer"
    rows = [(NS + "k_residue_small<false, 1>(oz2::Problem, unsigned int)", 64, 2000.0),
            (NS + "k_residue_gemm<false>(oz2::Problem)", 64, 3000.0),
            (NS + "void k_residue6<false, E2M3>(oz2::Problem, int)", 64, 4000.0),
            (NS + "k_residues6<false>(oz2::Problem, oz2::Group)", 64, 50000.0)]
    _counters(tmp_path / "f_counter_collection.csv", "FETCH_SIZE", [(copy, 1, 1048576.0)] + rows)
    _counters(tmp_path / "w_counter_collection.csv", "WRITE_SIZE", [(copy, 1, 1048576.0)] + rows)
    js = tmp_path / "t.json"
    ps.traffic(str(tmp_path), "f", "w", str(tmp_path / "t.md"), str(js))
    assert json.loads(js.read_text())["fetch_bytes_per_call"] == pytest.approx(9000.0 * 1024)


@pytest.mark.parametrize("which", range(3))
def test_the_hash_covers_every_product_source(tmp_path, monkeypatch, which):
    before = ps.gemm_source_sha()
    paths = list(ps.GEMM_SOURCES)
    changed = tmp_path / "changed.hip"
    changed.write_bytes(open(paths[which], "rb").read() + b"\n")
    paths[which] = str(changed)
    monkeypatch.setattr(ps, "GEMM_SOURCES", paths)
    assert ps.gemm_source_sha() != before
