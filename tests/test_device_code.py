"""Properties of the compiled device code that the sources rely on, read from the compiler's assembly (no GPU)."""
import subprocess

from paper_2606_00144_amd import build

MIXED = """
#include "bd_common.hpp"
#include "attn_tile.hpp"
__global__ void mixed(const uint16_t* g, uint32_t other, uint32_t off, float* o) {
  __shared__ __align__(16) uint8_t slot[8192];
  bd::dma16(g + threadIdx.x * 8, slot);
  HIDDEN;
  bd::dma16(g + threadIdx.x * 8 + 8192, slot);
  __syncthreads();
  o[threadIdx.x] = *reinterpret_cast<float*>(slot + 4 * threadIdx.x);
}
"""


def test_hidden_loads_leave_the_compilers_lds_base_alone(tmp_path):
    # A direct-to-LDS load that the compiler places takes its LDS base from M0, which it may keep over statements that
    # do not say that they write M0.  After a load issued by hand it has to set M0 again.
    for i, hidden in enumerate(["bd::dma16_hidden(g + threadIdx.x * 8 + 4096, other)",
                                "bd::dma16_hidden(g, off + 16 * threadIdx.x, other)"]):
        src, out = tmp_path / f"m{i}.hip", tmp_path / f"m{i}.s"
        src.write_text(MIXED.replace("HIDDEN", hidden))
        r = subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", str(src), "-o", str(out)],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        ops = [line.split()[:2] for line in out.read_text().splitlines() if "m0" in line or "global_load_lds" in line]
        bases = [op[1].rstrip(",") == "m0" for op in ops if op]
        # base, load | base, load (by hand) | base, load
        assert bases == [True, False] * 3, ops
