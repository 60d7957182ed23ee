"""The rank-r products of adapters over the sizes of their work-groups (8, 16 or 32 rows by 16, 8 or 4 wavefronts): rows
that do not fill one, either side of the sizes at which the choice changes, several problems in a launch, and contractions
with fewer chunks than wavefronts."""
import pytest

import synth_inputs as synth
from helpers import f64
from oracle.lora import layer_backward_reuse_lora
from test_gpu_lora import compare, make_case, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,rank", [(1, 8), (9, 16), (200, 64), (690, 8), (1370, 24), (2049, 8), (4100, 8)])
def test_rows_of_the_down_products(T, rank):
    lens = [min(61, T - a) for a in range(0, T, 61)]
    cu = synth.ragged_cu(lens)
    shp, osh, W, lora, lora64, rec, dY, scale = make_case("medium", "bf16", cu, 31, rank, synth.PROJECTIONS, record="drawn", dy_std=0.01)
    ref = layer_backward_reuse_lora(osh, cu, None, f64(rec), f64(W), lora64, scale, dY)
    gpu = run_gpu(shp, "bf16", cu, W, lora, rank, scale, rec, dY)
    compare({k: v for k, v in gpu.items()}, {k: ref[k] for k in gpu}, "bf16")


@pytest.mark.parametrize("T,rank", [(70, 16), (70, 32), (1400, 32), (2100, 16), (2100, 32)])
def test_four_groups_of_columns_go_round_their_rings(monkeypatch, T, rank):
    """Four groups of eight columns (rank 32, or gate and up of rank 16 in one pass) have the shortest rings, two to four stages
    a wavefront.  K 4096: 64 chunks, of which each of 16, 8 or 4 wavefronts takes 4, 8 or 16."""
    monkeypatch.setitem(synth.SHAPES, "wide", (4096 if rank == 16 else 256, 4, 2, 128, 256 if rank == 16 else 4096, 1e-5, 10000.0))
    lens = [min(61, T - a) for a in range(0, T, 61)]
    cu = synth.ragged_cu(lens)
    shp, osh, W, lora, lora64, rec, dY, scale = make_case("wide", "bf16", cu, 31, rank, synth.PROJECTIONS, record="drawn", dy_std=0.01)
    ref = layer_backward_reuse_lora(osh, cu, None, f64(rec), f64(W), lora64, scale, dY)
    gpu = run_gpu(shp, "bf16", cu, W, lora, rank, scale, rec, dY)
    compare({k: v for k, v in gpu.items()}, {k: ref[k] for k in gpu}, "bf16")
