"""The autotuner's walk over variants, on the host: whatever a variant's results are, the choice it ends with has
agreed with the reference, or is the reference."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_12089_amd", "csrc")

SRC = r"""
#include <cstdio>
#include <cstring>
#include <functional>
#include <vector>
#include "mpm_tune.h"
using mpmx::TuneChoice;

static bool same(const TuneChoice& a, const TuneChoice& b) { return !std::memcmp(&a, &b, sizeof a); }
static const TuneChoice kDefault{2, 1, 2, 1, 0, 1, 1, 1, 0, 0};

struct Outcome { TuneChoice best; int rc; bool sound; int tried; };

// agrees and ms stand in for the GPU; budget: attempts before over_budget, fail_at: attempt that errors
static Outcome walk(std::function<bool(const TuneChoice&)> agrees, std::function<double(const TuneChoice&)> ms,
                    int budget = 1000, int fail_at = -1) {
  std::vector<TuneChoice> good{mpmx::kTuneReference};
  int n = 0;
  Outcome o{};
  o.rc = mpmx::tune_choice(
      [&](const TuneChoice& c, bool, double& t, bool& ok) {
        if (n++ == fail_at) return 5;
        t = ms(c);
        ok = agrees(c);
        if (ok) good.push_back(c);
        return 0;
      },
      [&] { return n >= budget; }, o.best);
  for (const TuneChoice& c : good) o.sound |= same(c, o.best);
  o.tried = n;
  return o;
}

int main() {
  auto flat = [](const TuneChoice&) { return 1.0; };
  auto all = [](const TuneChoice&) { return true; };
  auto is_ref = [](const TuneChoice& c) { return same(c, mpmx::kTuneReference); };
  Outcome o = walk([](const TuneChoice&) { return false; }, flat);            // nothing agrees
  if (o.rc || !is_ref(o.best)) return 1;
  o = walk([](const TuneChoice& c) { return !c.fuse_adj; }, flat);            // a faulty adjoint pair
  if (o.rc || !o.sound || o.best.fuse_adj || o.best.p2g != 2 || o.best.g2p_adj != 2 || o.best.g2p != 1 || !o.best.fuse) return 2;
  o = walk([](const TuneChoice& c) { return c.g2p_adj == 0 && !c.fuse_adj; }, flat);   // a faulty G2P adjoint scatter
  if (o.rc || !o.sound || o.best.g2p_adj || o.best.fuse_adj || o.best.p2g != 2) return 3;
  o = walk([](const TuneChoice& c) { return c.g2p == 0; }, flat);             // a faulty gather
  if (o.rc || !o.sound || o.best.g2p) return 4;
  o = walk(all, flat);                                                        // ties keep the defaults
  if (o.rc || !same(o.best, kDefault)) return 5;
  o = walk(all, [](const TuneChoice& c) { return 10.0 - c.box - c.grid_list - 0.5 * c.xcd + (c.fuse == 0); });
  if (o.rc || o.best.box != 1 || o.best.grid_list != 2 || o.best.xcd != 1 || o.best.fuse != 1) return 6;
  o = walk([](const TuneChoice& c) { return c.box == 0; }, [](const TuneChoice& c) { return c.box ? 0.1 : 1.0; });
  if (o.rc || !o.sound || o.best.box) return 7;                               // the fastest does not agree
  o = walk(all, flat, 1);                                                     // no budget: the defaults, checked once
  if (o.rc || !same(o.best, kDefault) || o.tried != 1) return 8;
  for (int k = 0; k < 18; ++k) {                                              // an error at any attempt
    o = walk(all, [](const TuneChoice& c) { return 10.0 - c.box; }, 1000, k);
    if (o.rc != 5 || !o.sound) return 9;
  }
  // one option after another goes wrong: every subset of {p2g, g2p_adj, fuse, fuse_adj, box} that is off
  for (int m = 0; m < 32; ++m) {
    o = walk([m](const TuneChoice& c) {
      return !((m & 1 && c.p2g) || (m & 2 && c.g2p_adj) || (m & 4 && c.fuse) || (m & 8 && c.fuse_adj) || (m & 16 && c.box));
    }, flat);
    if (o.rc || !o.sound) return 10;
  }
  std::puts("ok");
  return 0;
}
"""


def test_the_choice_has_always_agreed(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "tune.cpp", tmp_path / "tune"
    src.write_text(SRC)
    subprocess.run([cxx, "-O1", "-std=c++17", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
