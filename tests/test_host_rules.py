"""What a CPU can check of the kernels' sources: arithmetic and rules of their headers, compiled for the host and run at sizes
that no test holds in memory, and the registers that the compiler gives a kernel."""
import os
import re
import subprocess

import pytest

import paper_1804_10112_amd as spt
from paper_1804_10112_amd import build as spt_build

INCLUDES = ["-I", spt_build.CSRC]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _run(tmp_path, text, stdin=""):
    src, exe = tmp_path / "check.hip", tmp_path / "check"
    src.write_text(text)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", *INCLUDES, str(src), "-o", str(exe)], check=True,
                   capture_output=True)
    return subprocess.run([str(exe)], check=True, input=stdin, capture_output=True, text=True, timeout=60).stdout


RANGES = r"""
#include <climits>
#include <vector>
#include "rows.hpp"
// Every element of l + 1 .. h once, and none beside them: what lies outside is counted, not stored, and the walk ends.
static bool whole(int l, int h) {
  std::vector<int> times(static_cast<size_t>(h - l), 0);
  long long outside = 0, steps = 0;
  for (int lane = 0; lane < spt::kWave; ++lane) {
    const auto one = [&](int r) {
      if (++steps > 100000) throw 1;
      const long long at = static_cast<long long>(r) - l - 1;
      if (at >= 0 && at < h - l) ++times[at]; else ++outside;
    };
    spt::wave_range(l, h, lane, [&](int r) { for (int q = 0; q < 4; ++q) one(r + q); }, one);
  }
  for (const int t : times) if (t != 1) return false;
  return outside == 0;
}
int main() {
  const int last[] = {0, 63, 300, INT_MAX - 600, INT_MAX - 257, INT_MAX - 256, INT_MAX - 65, INT_MAX - 64, INT_MAX - 2, INT_MAX - 1};
  const int length[] = {1, 17, 63, 64, 65, 254, 255, 256, 257, 511, 512, 513, 700, 1024};
  for (const int h : last)
    for (const int n : length)
      if (n <= h + 1) {  // l >= -1
        bool ok = false;
        try { ok = whole(h - n, h); } catch (int) {}
        if (!ok) { std::printf("(%d, %d]\n", h - n, h); return 0; }
      }
  std::printf("ok\n");
}
"""


def test_a_waves_share_of_pos_up_to_the_largest_row_counts(tmp_path):
    assert _run(tmp_path, RANGES) == "ok\n"


STRIDED = r"""
#include <climits>
#include <vector>
#include "common.hpp"
int main() {
  const int ends[] = {0, 1, 255, 256, 257, 100000, INT_MAX - 300, INT_MAX - 256, INT_MAX - 255, INT_MAX - 2, INT_MAX - 1};
  const int lengths[] = {0, 1, 63, 64, 65, 255, 256, 257, 1000};
  for (const int hi : ends)
    for (const int n : lengths) {
      if (n > hi) continue;
      std::vector<int> times(n, 0);
      int others = 0, calls = 0;
      for (int first = 0; first < 256 && calls < 100000; ++first)
        spt::strided(hi - n, hi, first, 256, [&](int r) {
          const long long at = static_cast<long long>(r) - (hi - n);
          if (++calls > 100000) std::abort();
          if (at >= 0 && at < n) ++times[at]; else ++others;
        });
      for (const int t : times) others += t != 1;
      if (others) { std::printf("[%d, %d)\n", hi - n, hi); return 0; }
    }
  std::printf("ok\n");
}
"""


def test_walks_over_rows_and_fibres_up_to_the_largest_numbers(tmp_path):
    assert _run(tmp_path, STRIDED) == "ok\n"


RULE = r"""
#include "slices.hpp"
int main() {
  long long nnz, x;
  int value, csr;
  while (std::scanf("%lld %lld %d %d", &nnz, &x, &value, &csr) == 4)
    std::printf("%d\n", value == 8 ? spt::slices_of_many<double>(nnz, x / 8, csr) : spt::slices_of_many<float>(nnz, x / 4, csr));
}
"""


def test_more_entries_to_a_lane_only_where_they_save_looks(tmp_path):
    """A round of the chip is 1024 * 256 lanes. With no round saved, the kernel of more entries only looks at more registers;
    with looks saved, it is the faster one from x of 12 MB on."""
    cases = [(n, x, v, csr) for n in range(16_800_000, 120_000_000, 100_001) for x in (6_500_000, 20_000_000, 30_000_000, 64_000_000)
             for v in (4, 8) for csr in (0, 1)]
    got = _run(tmp_path, RULE, "\n".join("%d %d %d %d" % c for c in cases)).split()
    assert len(got) == len(cases)
    for (n, x, v, csr), many in zip(cases, got):
        entries = 40 if v == 8 else 64
        few, more = (-(-n // (1024 * 256 * e)) for e in (32, entries))
        if few == more:
            assert many == "0", (n, x, v, csr)
        elif more * entries < few * 32 and x > 12_000_000:
            assert many == "1", (n, x, v, csr)
        elif v == 8 and more * entries > few * 32 * 1.1:
            assert many == "0", (n, x, v, csr)


@pytest.mark.parametrize("fmt", ["coo", "csf"])
@pytest.mark.parametrize("dtype,J", [("f64", 32), ("f32", 64), ("f64", 16), ("f32", 32)])
def test_mttkrp_has_more_workgroups_than_compute_units(fmt, dtype, J):
    """Carries and bounds of a workgroup take 16 bytes and a row. A tensor that more than one workgroup on each of 256
    compute units holds has no fewer than four for three of them: with about as many as compute units, the last decides."""
    def workgroups(nnz):
        t = spt.binding.SptTensor()
        t.order, t.nlevels, t.dtype, t.vals, t.nvals = 3, 3, spt.SPT_F64 if dtype == "f64" else spt.SPT_F32, 0x1000, nnz
        for k, lv in enumerate(t.level[:3]):
            csf = fmt == "csf"
            lv.kind, lv.mode, lv.N, lv.crd, lv.crd_stride = 1 if csf or k == 0 else 2, k, 1000, 0x1000, 1
            lv.M, lv.pos = (1, 0x1000) if k == 0 else (100, 0x1000) if csf else (0, None)
            lv.flags = spt.SPT_ORDERED | (spt.SPT_UNIQUE if csf or k == 2 else 0)
        row = J * (8 if dtype == "f64" else 4)
        return spt.spt_workspace_bytes(spt.SPT_OP_MTTKRP, t, J) / (16 + row + (4 + row) / 64)
    for nnz in range(200_000, 3_000_000, 1001):
        assert workgroups(nnz) > 340, (nnz, workgroups(nnz))


PARTS = r"""
#include <vector>
#include "mttkrp_plan.hpp"
int main() {
  long long nnz, J, rows_c, rows_d;
  int dtype, csf;
  while (std::scanf("%lld %lld %lld %lld %d %d", &nnz, &J, &rows_c, &rows_d, &dtype, &csf) == 6) {
    const int value = dtype == SPT_F64 ? 8 : 4;
    const int parts = spt::mttkrp_parts(nnz, J * value, rows_c, rows_d, csf);
    const spt::MttkrpPlan P = spt::mttkrp_plan(nnz, J, dtype, csf, parts);
    std::vector<int> kept(J, 0), of_part(parts, 0);
    int outside = 0;
    for (int part = 0; part < parts; ++part)
      for (int v = 0; v < P.tiles * P.lanes; ++v) {
        bool keeps;
        const int col = spt::column_of(static_cast<int>(J) / parts, P.vec, part, v, &keeps);
        outside += col < 0 || col + P.vec > J;
        for (int x = 0; keeps && x < P.vec; ++x)
          if (col + x < J) of_part[part] += kept[col + x]++ == 0;
      }
    int missed = 0, least = of_part[0], most = of_part[0];
    for (const int k : kept) missed += k == 0;
    for (const int n : of_part) least = std::min(least, n), most = std::max(most, n);
    std::printf("%d %d %d %d %d %d\n", parts, outside, missed, least, most, parts * P.tiles * P.lanes * P.vec);
  }
}
"""


def test_parts_of_the_columns_are_equal_and_cover_them(tmp_path):
    """Workgroups of every part have as many columns, of whole lines, and no more than a quarter of their lanes idle."""
    cases = [(n, J, c, d, dtype, csf) for n in (200_000, 20_000_000) for J in range(1, 1025) for c, d in ((20_000, 10_000), (4000, 4000), (9000, 9000))
             for dtype in (spt.SPT_F64, spt.SPT_F32) for csf in (0, 1)]
    got = _run(tmp_path, PARTS, "\n".join("%d %d %d %d %d %d" % c for c in cases)).splitlines()
    assert len(got) == len(cases)
    several = set()
    for (n, J, c, d, dtype, csf), line in zip(cases, got):
        parts, outside, missed, least, most, lanes = map(int, line.split())
        assert outside == 0 and missed == 0 and least == most == J // parts, (n, J, c, d, dtype, csf, line)
        if parts > 1:
            assert J // parts * (8 if dtype == spt.SPT_F64 else 4) % 128 == 0 and 4 * J >= 3 * lanes, (n, J, c, d, dtype, csf, line)
            several.add((J, dtype, parts))
    assert {(96, spt.SPT_F64, 2), (192, spt.SPT_F64, 4), (640, spt.SPT_F64, 4), (768, spt.SPT_F32, 8)} <= several


def _scratch(tmp_path, source, kernel):
    """Bytes of scratch memory of the kernels of a name."""
    asm = tmp_path / "kernels.s"
    flags = [f for f in spt_build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run([HIPCC, *flags, "--offload-device-only", "-S", os.path.join(spt_build.CSRC, source), "-o", str(asm)],
                   check=True, capture_output=True)
    return dict(re.findall(rf"\.name:\s+(\S*{kernel}\S*)\s+\.private_segment_fixed_size: (\d+)", asm.read_text()))


def test_the_kernel_that_gathers_slice_by_slice_keeps_its_registers(tmp_path):
    """Entries of a lane take 80 of its 128 registers; what no longer fits beside them would go through scratch memory."""
    scratch = _scratch(tmp_path, "spmv_slices.hip", "slices_spmv_kernel")
    assert len(scratch) == 8 and set(scratch.values()) == {"0"}, scratch


def test_mttkrp_keeps_its_registers(tmp_path):
    """Five waves a SIMD are asked for only where what a lane holds fits."""
    scratch = _scratch(tmp_path, "mttkrp.hip", "mttkrp_rows_kernel")
    assert len(scratch) > 70 and set(scratch.values()) == {"0"}, {k: v for k, v in scratch.items() if v != "0"}
