"""The launch plan of an attention call (csrc/plan.h), compiled for the CPU and walked over batches, heads, widths, window
sizes and lengths: every plan has to be one that the launch accepts and the workspace holds.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <stdio.h>
#include <stdlib.h>
#include "paper_2602_23200_amd/csrc/plan.h"
using namespace innerq;

static size_t workspace_of(const innerq_config_t& c) {           // innerq_workspace_bytes
  return seq_bytes(c) + (size_t)c.batch * c.n_q_heads * ((size_t)split_cap(c) + window_chunk_cap(c)) * (kHeadDim + 2) * sizeof(float) + 64;
}

int main() {
  const int heads[] = {1, 2, 3, 4, 5, 8, 13, 32, 64, 65, 112, 256, 320, 1024, 2100}, rs[] = {1, 4, 5, 8}, widths[][2] = {{2, 2}, {3, 2}, {3, 3}, {4, 4}};
  const int recents[] = {1, 2, 32, 128, 900, 2000, 6144, 6700, 8192, 16384, 40000};
  long long plans = 0, joined = 0, bad = 0;
  for (int bh : heads) for (int r : rs) for (auto& w : widths) for (int group = 32; group <= 64; group += 32) for (int recent : recents) {
    innerq_config_t c = {};
    c.batch = bh; c.n_kv_heads = 1; c.n_q_heads = r; c.head_dim = 128; c.bits = w[0]; c.v_bits = w[1]; c.group = group;
    c.w_sink = 4; c.w_recent = recent; c.capacity_tokens = 1 << 20;
    for (long long n_both = 0; n_both <= 140000; n_both = n_both < 40000 ? n_both + 3 * group : n_both * 9 / 8 / group * group)
      for (int kind = 0; kind <= 3; ++kind) for (int form = 0; form < 4; ++form) {
        if (kind != kInnerKernel && form > 0) continue;
        PlanInput in = {};
        in.fused_kind = kind; in.compute_units = 256; in.waves_per_cu = 8;
        in.may_join = kind == kInnerKernel; in.appends = form == 1 || form == 3; in.ragged = form == 2; in.spills = form == 3;
        in.n_both = in.ragged && n_both < 64 ? 64 : n_both;
        in.win_tokens = c.w_sink + recent + (n_both / group) % 2 * (group - 1);
        const LaunchPlan p = plan_attention(c, in);
        ++plans;
        joined += p.joins;
        const char* why = nullptr;
        if (p.workspace_bytes > workspace_of(c)) why = "workspace";
        if (p.n_win > window_chunk_cap(c) || (long long)p.n_win * kWindowChunk < in.win_tokens) why = "window chunks";
        if (in.n_both > 0 && p.n_splits < 1) why = "no wavefront";
        if (kind == kInnerKernel && in.n_both > 0) {
          if (p.waves < 1 || p.waves > kJoinWaves) why = "wavefronts of a work-group";
          if (!p.joins && p.waves > 1 && (r <= 4 || in.ragged)) why = "wavefronts that no kernel is built for";
          if (p.n_splits <= p.n_win) why = "no wavefront without a window chunk";
          if (p.joins && bh < 4 * in.compute_units && (long long)bh * p.n_partials > in.compute_units * (8 / p.waves)) why = "joined in more than one round";
          if (p.joins && in.spills && bh < in.compute_units) why = "joined although a value group leaves";
          if (p.joins && (p.n_splits != p.n_partials * p.waves || p.n_partials > kJoinGroups)) why = "joined launch";
          if (p.shared_groups && (p.joins || c.batch > kSharedBatchMost || (long long)(p.n_win + 1) * c.batch > p.shared_groups)) why = "shared wavefronts";
        } else if (p.joins || p.shared_groups || p.waves != 1) {
          why = "a plan of the inner kernel's";
        }
        if (why && ++bad <= 10)
          printf("%s: %d heads, r %d, %d/%d bits, G %d, w_recent %d, n_both %lld, kernel %d, form %d: %d wavefronts, %d chunks, %d partials\n",
                 why, bh, r, w[0], w[1], group, recent, in.n_both, kind, form, p.n_splits, p.n_win, p.n_partials);
      }
  }
  printf("%lld plans, %lld joined, %lld bad\n", plans, joined, bad);
  return bad || joined * 40 < plans;
}
"""

GRIDS = r"""
#include <stdio.h>
#include <initializer_list>
#include "paper_2602_23200_amd/csrc/plan.h"
using namespace innerq;

int main() {
  long long bad = 0, most = 0;
  for (long long recent : {32LL, 4096LL, 500000LL, 1048000LL, 1100000LL, 5000000LL, 16000000LL}) for (int n_both : {32, 64, 4096}) for (int tile = 64; tile <= 128; tile *= 2) {
    innerq_config_t c = {};
    c.batch = 1; c.n_kv_heads = 1; c.n_q_heads = 1; c.head_dim = 128; c.bits = tile == 64 ? 4 : 2; c.group = 32; c.w_sink = 4;
    c.w_recent = (int)recent; c.capacity_tokens = 1 << 24; c.kind = INNERQ_KIND_OUTER;
    PlanInput in = {};
    in.fused_kind = kOuterKernel; in.compute_units = 256; in.waves_per_cu = 8; in.n_both = n_both; in.win_tokens = c.w_sink + recent; in.tile_tokens = tile;
    const LaunchPlan p = plan_attention(c, in);
    const long long parts = (long long)p.n_splits + p.n_win;
    most = parts > most ? parts : most;
    const HeadsByParts g = heads_by_parts(1, parts);
    if (g.y > 65536 || g.z > 65536 || (long long)g.y * g.z < parts || (g.z > 1 && g.y != kGridParts) || (parts <= kGridParts && g.z != 1)) ++bad;
  }
  printf("%lld parts at most, %lld bad\n", most, bad);
  return bad || most <= 65536;
}
"""


def run(tmp_path, text):
    gxx = shutil.which("g++") or shutil.which("clang++")
    if not gxx:
        pytest.skip("no C++ compiler")
    (tmp_path / "grids.cpp").write_text(text)
    exe = str(tmp_path / "grids")
    subprocess.run([gxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", ROOT, str(tmp_path / "grids.cpp"), "-o", exe], check=True)
    return subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=100)


def test_grids_of_long_windows(tmp_path):
    """The outer-grouped kernel's parts of a sequence-head (window chunks and token ranges) fit a grid's dimensions of 65536 each."""
    done = run(tmp_path, GRIDS)
    assert done.returncode == 0, done.stdout


def test_every_plan_can_be_launched(tmp_path):
    gxx = shutil.which("g++") or shutil.which("clang++")
    if not gxx:
        pytest.skip("no C++ compiler")
    src = tmp_path / "plans.cpp"
    src.write_text(MAIN)
    exe = str(tmp_path / "plans")
    subprocess.run([gxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", ROOT, str(src), "-o", exe], check=True)
    done = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=100)
    assert done.returncode == 0, done.stdout
