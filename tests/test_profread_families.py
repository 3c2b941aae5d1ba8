"""Kernel names of a trace and the library's own records give the same families, for every
kernel of the plain method."""
import os
import re

import pytest

from paper_2404_09213_amd import profread

SRC = os.path.join(os.path.dirname(os.path.abspath(profread.__file__)), "csrc", "qsv.hip")


@pytest.mark.parametrize("signature,family", [
    ("void k_pg_apply<HIP_vector_type<float, 2u> >(HIP_vector_type<float, 2u>*, int)", "k_pg_apply"),
    ("void k_pg_apply_one<HIP_vector_type<double, 2u> >(HIP_vector_type<double, 2u>*, int)", "k_pg_apply"),
    ("void k_pg_apply_vec<true, false>(HIP_vector_type<float, 2u>*, int)", "k_pg_apply"),
    ("void k_pg_adj_vec<true>(HIP_vector_type<float, 2u>*, int)", "k_pg_adj"),
    ("void k_pg_adj<HIP_vector_type<double, 2u> >(HIP_vector_type<double, 2u>*, int)", "k_pg_adj"),
    ("void k_coef<float, false>(CoefIn, int)", "k_coef"),
    ("void k_grad_reduce<64, 1>(double const*)", "k_grad_reduce"),
    ("k_pg_apply.sign", "k_pg_apply"),
])
def test_family(signature, family):
    assert profread._base(profread.short(signature)) == family


def test_every_plain_kernel_has_a_family():
    with open(SRC) as f:
        names = set(re.findall(r"\bk_pg_\w+(?=\()", f.read())) - {"k_pg_adj", "k_pg_apply"}
    assert names and {profread._base(n) for n in names} <= {"k_pg_adj", "k_pg_apply"}
