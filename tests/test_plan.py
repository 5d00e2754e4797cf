"""The launch planning of a verify pass (csrc/plan.h) on the host, without a
GPU: GEMM shapes and workspace layout over models and block sizes that the
library takes, at 256 compute units."""
import ctypes
import subprocess

import numpy as np
import pytest

from paper_2510_13161_amd import build, msd, synth

SHIM = r"""
#include "plan.h"
using namespace msd;
// blocks [n][4] (batch, n_slots, kappa, capacity) -> out [n][2 + 5 * 8]: workspace bytes, whether the static
// scratch holds the block, and the shapes of its QKV, O, FFN up, FFN down and head GEMMs
extern "C" void plan_blocks(const msd_model_config* cfg, const int32_t* blocks, int64_t n, int64_t* out) {
  PlanInputs in;
  in.cfg = *cfg;
  plan_rows(&in);
  for (int64_t i = 0; i < n; ++i) {
    const int32_t* b = blocks + 4 * i;
    const Layout L = layout(&in, b[0], b[1], b[2], b[3]);
    *out++ = (int64_t)L.total;
    *out++ = fits_static(L) ? 1 : 0;
    for (const GemmShape* g : {&L.s.qkv, &L.s.o, &L.s.up, &L.s.down, &L.s.head})
      for (int v : {g->n_tiles, g->K, g->splits, g->waves, g->jt, g->wg_tiles, g->row_groups, g->split_from})
        *out++ = v;
  }
}
"""

MODELS = {"tiny": synth.TINY, "0.6b": synth.DRAFT06B, "14b": synth.QWEN14B, "66b": synth.OPT66B,
          # the head whose last dispatch round is split, over a ragged vocabulary
          "ragged": synth.ModelShape("ragged", 1, 1024, 8, 2, 128, 1024, 148240, norm="layer"),
          # a small head at one row tile; a wide ungated FFN
          "gqa": synth.ModelShape("gqa", 4, 1024, 16, 4, 64, 2048, 16000),
          "wide": synth.ModelShape("wide", 4, 10240, 80, 8, 128, 40960, 250000, norm="layer", act="relu")}
MAX_ROWS = 144


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "shim.hip", d / "libplan.so"
    src.write_text(SHIM)
    subprocess.run([build.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-I" + build.INCLUDE,
                    "-I" + build.CSRC, "-o", str(lib), str(src)], check=True)
    fn = ctypes.CDLL(str(lib)).plan_blocks

    def run(model, blocks):
        b = np.ascontiguousarray(blocks, np.int32)
        out = np.empty((len(b), 42), np.int64)
        fn(ctypes.byref(msd.config_of(MODELS[model])), b.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(len(b)),
           out.ctypes.data_as(ctypes.c_void_p))
        return out
    return run


KAPPAS = (1, 4, 8, 13, 32)
CAPACITIES = (64, 256, 300, 1024, 2048, 4096, 8192, 32768)


@pytest.mark.parametrize("model", sorted(MODELS))
def test_gemm_shapes_depend_on_the_row_tiles_alone(plan, model):
    """The kernels that a block runs, and with them the order of its sums, are
    the same whatever the early-exit width and the cache's capacity are, and
    however its rows are dealt over sequences."""
    blocks = [(b, n, k, c) for n in (1, 2, 5, 9, 16, 25, 33, 64) for b in range(1, MAX_ROWS // n + 1)
              for k in KAPPAS for c in CAPACITIES]
    out = plan(model, blocks)
    seen = {}
    for (b, n, k, c), row in zip(blocks, out[:, 2:]):
        first = seen.setdefault((b * n + 15) // 16, row)
        assert np.array_equal(first, row), (model, b, n, k, c)
    assert len(seen) == 9


@pytest.mark.parametrize("model", sorted(MODELS))
def test_early_exit_entry_point_runs_in_the_verify_workspace(plan, model):
    """msd_early_exit_topk lays out its rows as one sequence in a cache of one
    position: never more than a verify pass of as many rows needs."""
    for n in (1, 2, 5, 9, 16, 25, 33, 64):
        batches = range(1, MAX_ROWS // n + 1)
        for k in KAPPAS:
            own = plan(model, [(1, b * n, k, 1) for b in batches])[:, 0]
            for c in CAPACITIES:
                verify = plan(model, [(b, n, k, c) for b in batches])[:, 0]
                assert (own <= verify).all(), (model, n, k, c, np.argmax(own > verify) + 1)


@pytest.mark.parametrize("model", sorted(MODELS))
def test_workspace_never_falls_with_a_larger_block(plan, model):
    """A workspace for the largest block serves every smaller one: the size
    does not fall with batch, slots, early-exit width or capacity (up to
    blocks of more rows than a verify pass takes, which acceptance takes)."""
    batches, slots = range(1, MAX_ROWS + 9), (1, 2, 3, 5, 8, 9, 16, 17, 25, 33, 48, 49, 63, 64)
    grid = [(b, n, k, c) for b in batches for n in slots for k in KAPPAS for c in CAPACITIES]
    t = plan(model, grid)[:, 0].reshape(len(batches), len(slots), len(KAPPAS), len(CAPACITIES))
    for axis in range(4):
        assert (np.diff(t, axis=axis) >= 0).all(), (model, ("batch", "slots", "kappa", "capacity")[axis])


@pytest.mark.parametrize("model", sorted(MODELS))
def test_static_scratch_holds_what_its_documented_size_holds(plan, model):
    blocks = [(b, n, k, c) for n in (1, 2, 5, 9, 16, 25, 33, 64) for b in range(1, MAX_ROWS // n + 1)
              for k in KAPPAS for c in CAPACITIES]
    out = plan(model, blocks)
    small = out[:, 0] <= msd.MSD_STATIC_SCRATCH_BYTES
    assert small.any() and (out[small, 1] == 1).all()


# at the bound of the static scratch: blocks that fit it, without and with split partials past it
@pytest.mark.parametrize("model,block,fits", [
    ("0.6b", (15, 9, 4, 64), 1), ("0.6b", (16, 9, 4, 64), 1), ("0.6b", (16, 9, 8, 64), 1), ("0.6b", (127, 1, 8, 256), 1),
    ("66b", (1, 33, 4, 2048), 1), ("66b", (2, 33, 1, 2048), 1), ("66b", (2, 33, 4, 2048), 1), ("66b", (8, 9, 1, 2048), 1),
    ("14b", (1, 9, 8, 1088), 1), ("14b", (1, 25, 4, 4160), 1), ("14b", (71, 1, 1, 8192), 1), ("14b", (16, 9, 1, 8192), 0),
    ("0.6b", (16, 9, 32, 64), 0), ("66b", (16, 9, 1, 2048), 0)])
def test_static_scratch_at_its_bound(plan, model, block, fits):
    assert plan(model, [block])[0, 1] == fits


@pytest.mark.parametrize("model,rows,splits", [("14b", 33, 6), ("14b", 49, 3), ("14b", 144, 3), ("ragged", 33, 4),
                                               ("ragged", 48, 4), ("ragged", 49, 3), ("ragged", 144, 3)])
def test_last_dispatch_round_of_the_head_is_split(plan, model, rows, splits):
    """The head of 33 rows and more over a large vocabulary: whole K in the full
    dispatch rounds, splits of K in the last one, for every early-exit width."""
    for kappa in KAPPAS:
        n_tiles, _, s, _, _, wg_tiles, _, split_from = plan(model, [(1, rows, kappa, 64)])[0, 2 + 4 * 8:]
        assert (s, wg_tiles) == (splits, 4) and 0 < split_from < n_tiles and split_from % 4 == 0
    assert model != "ragged" or n_tiles % 4 == 1
