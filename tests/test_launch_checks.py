"""What the matrix-core kernel's launcher refuses (CPU): requests that a kernel instance does not implement must come
back as an error before anything is launched, whatever the routing above it does.  A small host program calls the
launcher itself; a request that passes the checks gets as far as the runtime, which has another error for it where
there is no GPU (so the program only makes requests that have to be refused, and one that shows the difference)."""
import os
import subprocess

import pytest
import torch

import paper_2604_16957_amd as tq
from paper_2604_16957_amd import build

PROGRAM = r"""
#include <cstdio>
#include "tq_internal.h"
using namespace tq;
int main() {
  DecodeParams plain{};                     // 8 heads on one KV head, d = 128, 64 tokens in two chunks
  plain.out = reinterpret_cast<half_t*>(256);
  plain.n_q_heads = 8; plain.n_kv_heads = 1; plain.gqa = 8; plain.group = 32; plain.n_queries = 1; plain.kv_share = 1;
  plain.row_stride = 64; plain.seq_len = 64; plain.n_splits = 2; plain.tokens_per_split = 32; plain.batch = 1;
  auto ask = [](const char* what, const DecodeParams& p, int merge_slot) {
    std::printf("%s %d\n", what, (int)launch_partial_mfma(p, p.batch, 128, merge_slot, nullptr));
  };
  if (LAUNCH) ask("plain", plain, 0);
  DecodeParams p = plain;
  p.gqa = 16; p.n_q_heads = 16;             // sixteen rows to a tile: no chunk merge in the kernel
  ask("tile16_merge", p, 0);
  p.n_splits = 1; p.tokens_per_split = 64;  // 32 rows in two such tiles: they take no new token
  p.gqa = 32; p.n_q_heads = 32; p.kv_share = 2; p.k_new = p.v_new = reinterpret_cast<const half_t*>(256);
  ask("shared_tile_new_token", p, 0);
  DecodeParams m = plain;                   // more chunks than the in-kernel merge holds
  m.seq_len = m.row_stride = 32 * 65; m.n_splits = 65;
  ask("merge_of_65_chunks", m, 0);
  DecodeParams r = plain;                   // one chunk per row, blocks of one wave, two rows to a block
  r.n_splits = 1; r.tokens_per_split = 64; r.seq_lens = reinterpret_cast<const int32_t*>(256);
  r.ranked = 1; r.waves_per_row = 1; r.rank_spread = 0;
  ask("one_wave_two_rows", r, 0);
  DecodeParams l = plain;                   // waves dealt to the sequences: only with counters, a slot for each, one query token, no window
  l.seq_lens = reinterpret_cast<const int32_t*>(256); l.listed = 1; l.var_chunks = 2048;
  ask("listed_no_merge", l, -1);
  DecodeParams w = l;
  w.window = 32;
  ask("listed_window", w, 0);
  w = l; w.batch = 257;
  ask("listed_many", w, 0);
  w = l; w.gqa = 16; w.n_q_heads = 16; w.n_splits = 1;        // (one chunk: nothing else refuses a sixteen-row tile)
  ask("listed_tile16", w, 0);
  return 0;
}
"""
INVALID_VALUE = 1                            # hipErrorInvalidValue


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    where = tmp_path_factory.mktemp("launch_checks")
    (where / "ask.cpp").write_text(PROGRAM)
    lib = tq.library_path()
    launch = 0 if torch.cuda.is_available() else 1
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")] + [f"-DLAUNCH={launch}"]
    subprocess.run([build.HIPCC, *flags, str(where / "ask.cpp"), "-o", str(where / "ask"), f"-L{lib.parent}",
                    f"-l:{lib.name}", f"-Wl,-rpath,{lib.parent}"], check=True, capture_output=True)
    out = subprocess.run([str(where / "ask")], check=True, capture_output=True, text=True, env=dict(os.environ)).stdout
    return {line.split()[0]: int(line.split()[1]) for line in out.splitlines()}


def test_a_request_that_is_covered_gets_past_the_checks(answers):
    if "plain" in answers:                   # (no GPU here: the runtime refuses it, for another reason)
        assert answers["plain"] not in (0, INVALID_VALUE)


@pytest.mark.parametrize("request_", ["tile16_merge", "merge_of_65_chunks", "shared_tile_new_token", "one_wave_two_rows",
                                      "listed_no_merge", "listed_window", "listed_many", "listed_tile16"])
def test_a_request_no_instance_implements_is_refused(answers, request_):
    assert answers[request_] == INVALID_VALUE
