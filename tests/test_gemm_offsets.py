"""The offset table of the pairwise GEMM steps, replayed on the host: a stage
loads every table entry without a condition, four elements at a time where an
operand is contiguous along the contraction, so every load has to lie inside
the operand also past the end of a chunk."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2307_15034_amd", "csrc")

SOURCE = r"""
#include <cstdio>
#include <initializer_list>
#include "fno_gemm_offsets.h"

// Operand [rows][K] (K contiguous; of a contraction over several indices, an
// innermost run, whose extent is then a multiple of four): the chunks
// [kb, kb + klen) of its work-groups in stages of tk.
static int check(int rows, int K, int tk, int kchunk) {
  const long size = (long)rows * K;
  int bad = 0;
  for (int kb = 0; kb < K; kb += kchunk) {
    const int klen = K - kb < kchunk ? K - kb : kchunk;
    const int nst = (klen + tk - 1) / tk;
    for (int row = 0; row < rows; ++row)
      for (int i = 0; i < nst * tk; ++i) {
        const int e = fno::gemm_k_entry(i, klen);
        bad += e < 0 || e >= klen || (i < klen && e != i);
        if (K % 4 || i % 4) continue;
        // a quad: 4-aligned, whole, inside the operand
        const long off = (long)row * K + kb + e;
        bad += off % 4 != 0 || off + 3 >= size || e + 3 >= klen;
      }
  }
  if (bad) std::printf("rows %d K %d stage %d chunk %d: %d\n", rows, K, tk, kchunk, bad);
  return bad;
}

int main() {
  int bad = 0;
  for (int tk = 16; tk <= 32; tk += 16)
    for (int rows : {1, 16, 33, 64, 256})
      for (int K = 4; K <= 260; ++K)
        for (int kchunk : {tk, 2 * tk, 2048}) bad += check(rows, K, tk, kchunk);
  for (int K : {2048, 2052, 4100, 65535, 65540}) bad += check(1, K, 32, 2048);
  return bad != 0;
}
"""


def test_every_load_lies_inside_the_operand(tmp_path):
    src, exe = tmp_path / "replay.cpp", tmp_path / "replay"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout[:2000]


def test_the_kernel_fills_its_table_with_these_entries():
    text = open(os.path.join(CSRC, "fno_gemm.hip")).read()
    assert "cls_decode(g.c[CL_K], (uint32_t)(kb + gemm_k_entry(i, klen))" in text
