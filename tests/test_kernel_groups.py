"""The kernels in the sources, those that something launches, and the groups that the benchmark's
profile summaries sort them into."""
import glob
import os
import re

import bench

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2009_12663_amd", "csrc")
SOURCE = "\n".join(open(f).read() for f in sorted(glob.glob(os.path.join(CSRC, "*.h*"))))
CODE = re.sub(r"//[^\n]*", "", SOURCE)
CODE = re.sub(r"__launch_bounds__\((?:[^()]|\([^()]*\))*\)|__attribute__\(\((?:[^()]|\([^()]*\))*\)\)", "", CODE)
DEFINED = re.findall(r"__global__\s+void\s+(\w+)(?:<[^>]*>)?\(", CODE)
KERNELS = sorted(set(DEFINED))


def test_kernels_are_found():
    assert len(DEFINED) == CODE.count("__global__")
    assert {"reduce_partials", "gemm2_mfma", "lu_factor", "qtx_mfma", "dc_first", "smooth_tile"} <= set(KERNELS)


def test_every_kernel_is_launched():
    assert not [k for k in KERNELS if len(re.findall(rf"\b{k}\b", CODE)) <= DEFINED.count(k)]


def test_every_group_key_names_a_kernel():
    for key, _ in bench.KERNEL_GROUPS:
        assert any(key in k for k in KERNELS) or re.search(rf"struct {key};", SOURCE), key


def test_projection_sum_belongs_to_the_projection():
    name = "void (anonymous namespace)::reduce_partials<(anonymous namespace)::%s>(long, int, double const*, double*)"
    assert bench.group_of(name % "ProjectionSum") == "proj_QtX"
    assert bench.group_of(name % "ApplySum") == "apply_reduce"
    assert bench.group_of("reduce_z(long, int, int, int, float const*)") == "apply_reduce"
