"""The benchmark's list of vector kernels is the library's."""
import os
import re

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_vector_kernel_names():
    src = open(os.path.join(ROOT, "paper_2201_09004_amd/csrc/ops.cpp")).read()
    body = re.search(r"blas_name\(int op\) \{\s*static const char\* n\[\] = \{([^}]*)\}", src).group(1)
    assert bench.BLAS_OPS == re.findall(r'"(\w+)"', body)
