"""Index arithmetic of the passes, checked on the host: a small program compiled from
the library's own headers (host code only) walks the extreme accepted sizes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2209_11922_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def _run(tmp_path, body):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "probe.hip", tmp_path / "probe"
    src.write_text('#include <cstdio>\n#include "eife_grid.hpp"\nusing namespace eife;\nint main() {\n' + body + "\nreturn 0;\n}\n")
    flags = ["--offload-host-only", "-O1", "-std=c++17", "-w", f"-I{CSRC}", "-o", str(exe), str(src)]
    built = subprocess.run([HIPCC, *flags], capture_output=True, text=True, timeout=300)
    assert built.returncode == 0, built.stderr[-2000:]
    ran = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert ran.returncode == 0, ran.stdout[-2000:]


def test_32_bit_tiles_only_where_the_offsets_fit(tmp_path):
    """The passes that keep a tile's row offsets in 32 bits are taken only where the last
    element of a line lies less than 2^31 elements behind the first."""
    _run(tmp_path, """
  const int lens[] = {64, 128, 192, 256, 384, 512};
  int refused = 0;
  for (int n : lens)
    for (int n1 = 1; n1 <= 4096; ++n1)
      for (int pitch : {32, 1024, 4096}) {
        ColGeom cg{};
        cg.n = n;
        cg.ld_line = int64_t(pitch) * n1;
        const bool fits = tile_fits_32(cg);
        if (fits && int64_t(n) * cg.ld_line > 0x7fffffff) {
          printf("%d x %d x %d taken\\n", pitch, n1, n);
          return 1;
        }
        if (!fits && int64_t(n) * cg.ld_line <= 0x7fffffff) return 2;
        refused += !fits;
      }
  ColGeom cg{};  // 4096 x 2560 x 256 intervals: accepted, beyond 32 bits
  cg.n = 255;
  cg.ld_line = int64_t(4096) * 2559;
  if (tile_fits_32(cg) || refused == 0) return 3;
""")


def test_reactions_of_lines_past_the_end_stay_in_the_tables(tmp_path):
    """A row pass forms the reaction of every line of its blocks, up to 63 rows past the last one on
    odd row counts; the y and z indices it reads the forcing's tables at are those of rows."""
    _run(tmp_path, """
  Forcing F{};
  for (int ny : {1, 2, 63, 64, 511})
    for (int nz : {1, 3, 64, 255}) {
      RowGeom g{};
      g.ny = ny;
      g.nrows = ny * nz;
      for (int row = 0; row < g.nrows + 64; ++row) {
        const fast::RowReaction<float, fast::RK_GENERIC> r(F, g, row);
        if (r.iy < 0 || r.iy >= ny || r.iz < 0 || r.iz >= nz) {
          printf("row %d of %d x %d: %d, %d\\n", row, ny, nz, r.iy, r.iz);
          return 1;
        }
        if (row < g.nrows && r.iz * ny + r.iy != row) return 2;
      }
    }
""")
