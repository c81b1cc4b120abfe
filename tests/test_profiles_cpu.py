"""Figures from the committed rocprofv3 summaries appear in a bench line only beside the kernels they were read from."""
import bench
from paper_2603_09582_amd import build


def test_profile_figures_are_those_of_these_kernels(tmp_path, monkeypatch):
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    path = tmp_path / "profiles" / "binattn_kernels_w.txt"
    path.parent.mkdir()
    for text, want in [("traffic_bytes_per_launch: 8.9e9\n", None),
                       ("traffic_bytes_per_launch: 8.9e9\nkernel_source_id: 0123456789ab\n", None),
                       (f"traffic_bytes_per_launch: 8.9e9\nkernel_source_id: {build.kernel_source_id()}\n", 8.9e9)]:
        path.write_text(text)
        assert bench.profile_record("w") == want
    assert bench.profile_record("missing") is None


def test_source_id_follows_the_code_and_not_the_comments(tmp_path):
    f = tmp_path / "a.h"
    ids = []
    for text in ("int x = 1;  // one\n", "int x = 1; /* eins\n zwei */\n\n", "int x = 2;  // one\n"):
        f.write_text(text)
        ids.append(build.kernel_source_id([str(f)]))
    assert ids[0] == ids[1] != ids[2]
