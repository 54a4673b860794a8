"""Host memory of the RA/DEC conversion where pinned memory is refused: pageable
memory takes its place, pinned memory is tried again when more is wanted, and every
piece goes back the way it came (the header compiled on the CPU with stand-ins for
the two pinning calls)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <assert.h>
#include <stdio.h>
#include <string.h>
#include "pc_slabs.h"
static int refuse, pinned_now, pins, unpins;
static int pin(void **p, size_t n)
{
    if (refuse) { *p = nullptr; return 1; }
    pins++; pinned_now++;
    *p = malloc(n);
    return 0;
}
static int unpin(void *p) { unpins++; pinned_now--; free(p); return 0; }
int main()
{
    pc::HostSlabs s;
    refuse = 1;
    assert(s.grow(1000, pin, unpin) && s.data() && s.size() == 1000 && !s.pinned());
    memset(s.data(), 1, 1000);
    assert(s.grow(900, pin, unpin) && s.size() == 1000);
    refuse = 0;
    assert(s.grow(2000, pin, unpin) && s.pinned() && unpins == 0);
    memset(s.data(), 1, 2000);
    refuse = 1;
    assert(s.grow(3000, pin, unpin) && !s.pinned() && unpins == 1);
    memset(s.data(), 1, 3000);
    assert(!s.grow((size_t)1 << 62, pin, unpin) && !s.data() && s.size() == 0);
    assert(s.grow(10, pin, unpin) && !s.pinned());
    s.release(unpin);
    s.release(unpin);
    assert(!s.data() && pins == 1 && unpins == 1 && pinned_now == 0);
    puts("ok");
}
"""


def test_pageable_where_pinning_is_refused(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I",
                    os.path.join(ROOT, "paper_1911_03545_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout == "ok\n"
