"""Plans and layouts of the built library, computed on the CPU: the projection
planner (plan_gemm) and the workspace."""
import ctypes

import pytest

from paper_2609_37062_amd import vsk
from workloads.configs import M8B

RESID, QKV, SWIGLU, LOGITS = range(4)


class Plan(ctypes.Structure):
    """GemmPlan (csrc/gemm.hpp)."""
    _fields_ = [(n, ctypes.c_int) for n in ("mg", "m_tiles", "n_groups", "nt", "wn", "ksplit")] + \
        [("tiled", ctypes.c_bool), ("xl", ctypes.c_bool)]


def plan(N, K, R, epi, shape=0, resid_target=0, row_tile=0):
    f = vsk.lib()._ZN3vsk9plan_gemmEiiiiiii
    f.restype, f.argtypes = Plan, [ctypes.c_int] * 7
    return f(N, K, R, epi, shape, resid_target, row_tile)


@pytest.mark.parametrize("row_tile", [6, 7, 8, 11])
@pytest.mark.parametrize("rows", [129, 200, 405, 777, 2080])
@pytest.mark.parametrize("N,K", [(3072, 512), (4096, 1024), (1792, 4096), (16384, 3072), (28672, 4096)])
def test_forced_tile_height(N, K, rows, row_tile):
    """Key 10 forces the height of the gate/up tiles, however few the columns:
    eight waves side by side over 16 column tiles, as it is for wide ones."""
    p = plan(N, K, rows, SWIGLU, row_tile=row_tile)
    rg = (rows + 15) // 16
    assert p.xl and (p.mg, p.wn, p.nt) == (row_tile, 8, 2)
    assert (p.m_tiles, p.n_groups) == (-(-rg // row_tile), -(-N // 256))


@pytest.mark.parametrize("N,K,rows,tiles", [(3072, 512, 136, 2), (3072, 512, 600, 4), (3072, 512, 1150, 8),
                                            (1792, 4096, 256, 2), (16384, 3072, 200, 8), (28672, 4096, 777, 16)])
def test_automatic_gate_up_workgroups(N, K, rows, tiles):
    """Without key 10, gate/up of few columns takes narrower workgroups."""
    p = plan(N, K, rows, SWIGLU)
    assert p.nt * p.wn == tiles
    if tiles < 16:
        assert p.mg == 8


@pytest.mark.parametrize("N,K,rows,target,splits", [
    (1536, 512, 40, 4096, 2), (3072, 2048, 40, 256, 5), (3072, 2048, 40, 192, 4), (3072, 2048, 100, 192, 8),
    (3072, 2048, 100, 64, 3), (3072, 2048, 100, 128, 6), (3072, 2048, 100, 168, 7)])
def test_qkv_k_splits(N, K, rows, target, splits):
    """The split counts that the GPU tests of the QKV projection stand for: 2 to
    8, one for each count the reduction is compiled for."""
    assert plan(N, K, rows, RESID, resid_target=target).ksplit == splits


@pytest.mark.parametrize("rows,kv", [(256, 6001), (2080, 2048), (777, 777)])
def test_workspace_holds_what_a_pass_uses(rows, kv):
    """A workspace is the pass's buffers and their alignment, nothing beside them."""
    m = M8B
    splits = -(-(-(-kv // 16)) // 8) + 16                    # 8-block splits and prefix splits
    qkv = m.q_dim + 2 * m.kv_dim
    per_row = (4 * m.hidden                                  # residual
               + 2 * m.q_dim                                 # q
               + splits * m.n_q_heads * (4 * m.head_dim + 8) + 4 * m.n_kv_heads  # attention partials, arrivals
               + m.hidden // 16 * 8                          # sums of x^2
               + 8 * 4 * max(m.hidden, qkv)                  # products of K splits
               + m.vocab // 16 * 8)                          # argmax partials
    per_padded_row = 2 * m.q_dim + 2 * m.hidden + 2 * m.ffn  # projection inputs
    need = rows * per_row + -(-rows // 16) * 16 * per_padded_row
    e = vsk.Engine(m)
    assert need <= e.workspace_bytes(rows, 1, kv) <= need + 11 * 256
    e.close()
