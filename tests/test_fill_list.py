"""The list of buffers that one launch zeroes: more buffers than it holds are refused, with nothing
written past its slots and nothing launched.  A host program against the built library, no GPU needed."""
import os
import subprocess

from paper_2502_09323_amd import build as H

SRC = r"""
#include <cstdio>
#include <cstring>
#include "pb_internal.h"

int main()
{
    struct { unsigned char before[64]; pbk::FillList l; unsigned char after[64]; } s;
    std::memset(s.before, 0x5a, 64);
    std::memset(s.after, 0x5a, 64);
    static double buf[2];
    pbk::FillList ref;
    for (int k = 0; k < pbk::FillList::kMax; ++k) ref.add(buf, k + 1);
    s.l = ref;
    for (int k = 0; k < 40; ++k) s.l.add(buf + 1, 1000);
    for (int k = 0; k < 64; ++k)
        if (s.before[k] != 0x5a || s.after[k] != 0x5a) return 1;
    for (int k = 0; k < pbk::FillList::kMax; ++k)
        if (s.l.p[k] != buf || s.l.bytes[k] != k + 1) return 2;
    if (pbk::launch_fill(nullptr, s.l) != hipErrorInvalidValue) return 3;
    std::puts("ok");
    return 0;
}
"""


def test_more_buffers_than_slots_are_refused(tmp_path):
    if not os.path.exists(H.LIB):
        H.build()
    src, exe = tmp_path / "fill.hip", tmp_path / "fill"
    src.write_text(SRC)
    subprocess.run([H.hipcc(), "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(H.ROOT, "include"),
                    "-I", os.path.join(H.HERE, "csrc"), str(src), "-L", os.path.dirname(H.LIB), "-l:libpb.so",
                    f"-Wl,-rpath,{os.path.dirname(H.LIB)}",
                    "-o", str(exe)], check=True)
    p = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0 and p.stdout.strip() == "ok", (p.returncode, p.stdout, p.stderr)
