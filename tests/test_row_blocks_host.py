"""The packed (sequence, 32-row block) of a ragged prefill chunk, on the host: every
sequence of the largest batch and every block of the longest prompt comes back."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_row_blocks_come_back(tmp_path):
    src = tmp_path / "rows.hip"
    src.write_text('''#include <stdio.h>
#include "kernels.h"
int main() {
    const int ks[] = {0, 1, 255, 65535, 65536, 65537, 1 << 20, (1 << 26) - 1};   // 65536: position 2097152
    for (int b = 0; b < 64; ++b)
        for (int k : ks) {
            const uint32_t e = pipo::row_block(b, k);
            if (pipo::row_block_seq(e) != b || pipo::row_block_index(e) != k) { printf("%d %d\\n", b, k); return 1; }
        }
    return 0;
}''')
    exe = tmp_path / "rows"
    subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-I",
                    os.path.join(ROOT, "paper_2605_27255_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
