"""The HBM traffic figure of the benchmark's roofline belongs to the kernel that is built: host files only."""
import os

import pytest

import bench

PLAN = "attn_wave_kernel<128,8,2,1> workgroups=256 splits=1 merge_launch=0"
SOURCES = {"attn.hip": "int order(int i) { return i; }   // in the order of the keys\n", "common.h": "", "lds_tiles.h": "/* two\nlines */ int x;\n", "sizes.h": ""}


@pytest.fixture
def tree(tmp_path, monkeypatch):
    csrc = tmp_path / "paper_2505_19201_amd" / "csrc"
    csrc.mkdir(parents=True)
    (tmp_path / "profiles").mkdir()
    for name, text in SOURCES.items():
        (csrc / name).write_text(text)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    (tmp_path / "profiles" / "attn_verify_llava_traffic.txt").write_text(
        f"# a comment\ntraffic_bytes_per_launch: 13614596\nkernel: attn_wave_kernel<128,8,2,1>\nsources: {bench.attention_sources()}\nmeasured: 2026-12-04\n")
    return csrc


def test_a_figure_of_the_kernel_as_it_is(tree):
    traffic, source = bench.read_traffic("llava", PLAN)
    assert traffic == 13614596 and "2026-12-04" in source
    (tree / "attn.hip").write_text("int order(int i) {\n    return i;\n}\n// another comment, /* other blanks */\n")
    assert bench.read_traffic("llava", PLAN)[0] == 13614596


@pytest.mark.parametrize("name", sorted(SOURCES))
def test_a_figure_of_the_same_name_from_other_sources_is_stale(tree, name):
    (tree / name).write_text(SOURCES[name].replace("return i", "return i ^ 1") + "int y;\n")
    traffic, source = bench.read_traffic("llava", PLAN)
    assert traffic is None and "stale" in source


def test_a_figure_without_its_sources_or_of_another_kernel_is_stale(tree):
    assert bench.read_traffic("llava", PLAN.replace("<128,8,2,1>", "<128,8,4,1>"))[0] is None
    path = os.path.join(bench.ROOT, "profiles", "attn_verify_llava_traffic.txt")
    lines = [l for l in open(path) if not l.startswith("sources")]
    open(path, "w").writelines(lines)
    traffic, source = bench.read_traffic("llava", PLAN)
    assert traffic is None and "stale" in source
    assert bench.read_traffic("pixtral", PLAN) == (None, "no rocprofv3 summary committed for this configuration")
