"""bench.py names the kernel that ran, and prints counters of that kernel only."""
import pytest

import bench


@pytest.mark.parametrize("pattern,world,bf16,long_tiles,name", [
    ("ring", 8, False, True, "k_walk"), ("shuffle", 16, True, True, "k_walk"), ("ring", 6, False, False, "k_walk"),
    ("ring", 3, False, False, "k_walk"), ("ring", 1, False, False, "k_ring_reduce"), ("hd", 1, False, True, "k_walk"),
    ("ring", 8, False, False, "k_ring_reduce"), ("hd", 8, True, False, "k_ring_reduce"), ("hd", 8, False, True, "k_tree_walk"),
    ("hd", 16, True, True, "k_tree_walk"), ("hd", 32, False, True, "k_tree_walk"), ("hd", 64, True, True, "k_ring_reduce_tree_any"),
    ("hd", 32, False, False, "k_ring_reduce_tree_any")])
def test_name_of_the_reduce_kernel(pattern, world, bf16, long_tiles, name):
    assert bench.reduce_kernel(pattern, world, bf16, long_tiles) == name


@pytest.mark.parametrize("pattern,world,slices,name", [
    ("ring", 4, (263, 256, 1), "k_slice"), ("shuffle", 16, (256, 256, 12), "k_slices"), ("ring", 12, (256, 1024, 5), "k_slices"),
    ("hd", 1, (9, 256, 1), "k_slice"), ("hd", 8, (30, 256, 1), "k_tree_slice"), ("hd", 64, (200, 256, 8), "k_tree_slices"),
    ("ring", 8, None, "k_ring_reduce")])
def test_name_of_the_kernel_over_slices(pattern, world, slices, name):
    assert bench.reduce_kernel(pattern, world, False, False, slices) == name


def test_traffic_comes_from_a_profile_of_the_same_kernel(tmp_path, monkeypatch):
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    (tmp_path / "profiles").mkdir()
    f = tmp_path / "profiles" / "ring_reduce_vgg16_hbm_traffic.txt"
    f.write_text("HBM traffic of the ring-reduce kernel (k_walk<8, false, 2, 8>) on ...\ntraffic_bytes_per_launch: 8866879379\n")
    assert bench.read_traffic("vgg16", "k_walk") == 8866879379.0
    assert bench.read_traffic("vgg16", "k_tree_walk") is None
    assert bench.read_traffic("mlp", "k_ring_reduce") is None


def test_committed_profiles_are_of_the_kernel_that_runs():
    assert bench.read_traffic("vgg16", bench.reduce_kernel("ring", 8, False, True)) is not None
    assert bench.read_traffic("inception_v3", bench.reduce_kernel("ring", 16, False, True)) is not None
