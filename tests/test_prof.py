"""Which dispatches of a profile belong to a draft variant's projections, and when a kept profile is out of date."""
import pytest

import bench
from paper_2609_21704_amd import prof

INT4 = ["sq::gemv_kernel<1, false, 2>", "sq::gemv_rows_kernel<2, false, true>", "sq::tile_kernel<0, 1, 2, 8>",
        "sq::linear_kernel<0, 8, 1, false>", "sq::linear_kernel<0, 8, 2, true>"]
FP8 = ["sq::gemv_kernel<1, true, 2>", "sq::gemv_rows_kernel<4, true, false>", "sq::tile_kernel<1, 1, 1, 8>",
       "sq::linear_kernel<1, 8, 1, false>"]
OTHER = ["sq::tile_kernel<2, 1, 2, 8>", "sq::linear_kernel<2, 8, 3, false>", "sq::gemm_rows_kernel<5, 2>",
         "sq::prefill_gemm_kernel<0, 128, true>", "sq::accept_kernel<false, true>", "sq::slice_reduce_kernel<4, 0>"]


def test_draft_dispatches_of_each_variant():
    for names, variant in ((INT4, "int4"), (FP8, "fp8")):
        for name in INT4 + FP8 + OTHER:
            assert prof.is_draft_gemv(name, variant) == (name in names), (name, variant)


@pytest.mark.parametrize("variant,kind", [("int4", 0), ("fp8", 1)])
def test_draft_values_take_the_reductions_of_their_own_slices(variant, kind):
    reduce, split = "sq::slice_reduce_kernel<4, 1>", "sq::splitk_reduce_kernel<false>"
    own, verify = f"sq::linear_kernel<{kind}, 8, 2, false>", "sq::linear_kernel<2, 8, 2, false>"
    rows = [(own, 1), (reduce, 2), (reduce, 4), (verify, 8), (reduce, 16), (own, 32), ("sq::silu_mul_kernel", 64),
            (split, 128), (f"sq::gemv_kernel<2, {'true' if kind else 'false'}, 2>", 256), (split, 512)]
    assert sum(prof.draft_values(rows, variant)) == 1 + 2 + 32 + 256 + 512


def test_a_profile_is_kept_for_the_sources_that_hold_or_choose_the_kernels(tmp_path, monkeypatch):
    for f in ("gemv.hip", "gemm.hip", "linear.hip", "sq_internal.hpp"):
        assert f in prof.GEMV_SOURCES
    (tmp_path / "profiles").mkdir()
    path = tmp_path / "profiles" / "gemv_fp8_traffic.txt"
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    path.write_text(f"hbm_bytes_per_launch = 5.5\ngemv_source_sha256 = {prof.sources_sha()}\n")
    assert bench.traffic_from_profile("fp8") == 5.5
    path.write_text("hbm_bytes_per_launch = 5.5\ngemv_source_sha256 = 00\n")
    assert bench.traffic_from_profile("fp8") is None
