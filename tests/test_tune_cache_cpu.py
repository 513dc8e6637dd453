"""The tuner's file across builds: choices that were timed on earlier kernels
are not taken up."""
import pytest

prs = pytest.importorskip("paper_1710_10420_amd.prs")


@pytest.mark.parametrize("shape,key", [((64, 64), "2D|64x64x1"), ((64, 48, 32), "3D|64x48x32")])
def test_entries_of_earlier_kernels_are_not_found(tmp_path, shape, key):
    """k4: before the 2D block passes, the five-step pass and the LDS reverse
    passes, whose settings a found entry would keep from being used."""
    path = tmp_path / "tune.json"
    entry = '{"vec": 1, "rows": 32, "ty": 1, "steps_per_pass": 2, "us": 9.000}'
    path.write_text("{\n" + ",\n".join('"%s|%s|%s|k4": %s' % (arch, key, kind, entry)
                                       for arch in ("unknown", "gfx950") for kind in ("single", "batch")) + "\n}\n")
    for flags in (0, prs.PRS_TUNE_BATCH):
        assert prs.prs_tuned_tiling(prs.make_params(shape, deta=0.1), str(path), flags) is None
