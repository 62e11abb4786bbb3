"""Helpers and lists shared by the GPU parity tests: upload seeded inputs, run the oracle, compare."""
from __future__ import annotations

import numpy as np
import torch

import oracle
import paper_2405_18047_amd as tbp
import seeded_inputs as si

DEV = "cuda:0"

# (layout, (M, N, K), (tile rows, tile columns, workgroups per compute unit, slices)): storage-type products for every tile of the bf16 product
# plan, whole and (but for 32 x 32) in slices that end in a shorter one, in both layouts
PRODUCT_TILES = [
    (tbp.NN, (136, 1032, 2760), (32, 32, 1, 1)), (tbp.NT, (8, 4104, 4104), (32, 32, 1, 1)),
    (tbp.NN, (16, 8904, 8), (64, 64, 2, 1)), (tbp.NT, (16, 8648, 72), (64, 64, 2, 1)), (tbp.NN, (328, 920, 2808), (64, 64, 2, 2)),
    (tbp.NN, (24, 80, 2408), (64, 64, 2, 8)), (tbp.NT, (16, 72, 4720), (64, 64, 2, 15)),
    (tbp.NN, (408, 2352, 512), (128, 64, 1, 1)), (tbp.NT, (2832, 328, 464), (128, 64, 1, 1)), (tbp.NN, (584, 520, 2800), (128, 64, 1, 5)),
    (tbp.NT, (1912, 144, 2520), (128, 64, 1, 5)), (tbp.NT, (456, 664, 2456), (128, 64, 1, 5)),
    (tbp.NN, (400, 4760, 64), (128, 128, 2, 1)), (tbp.NN, (416, 8440, 64), (128, 128, 2, 1)), (tbp.NN, (1744, 3488, 800), (128, 128, 2, 1)),
    (tbp.NT, (392, 8952, 64), (128, 128, 2, 1)), (tbp.NT, (456, 8200, 720), (128, 128, 2, 1)), (tbp.NN, (136, 5872, 4120), (128, 128, 2, 5)),
    (tbp.NT, (2024, 72, 8016), (128, 128, 2, 16)),
    (tbp.NN, (144, 8344, 3112), (128, 128, 1, 1)), (tbp.NN, (3640, 520, 72), (128, 128, 1, 1)), (tbp.NT, (2312, 872, 72), (128, 128, 1, 1)),
    (tbp.NT, (136, 8608, 3376), (128, 128, 1, 1)), (tbp.NN, (16, 3280, 5264), (128, 128, 1, 8)), (tbp.NT, (72, 3424, 2792), (128, 128, 1, 5)),
    (tbp.NT, (408, 2976, 4040), (128, 128, 1, 2)),
    (tbp.NN, (1040, 3744, 320), (128, 192, 1, 1)), (tbp.NT, (2440, 1640, 960), (128, 192, 1, 1)), (tbp.NN, (288, 3928, 4000), (128, 192, 1, 4)),
    (tbp.NN, (168, 5904, 4416), (128, 192, 1, 4)), (tbp.NT, (152, 5936, 5056), (128, 192, 1, 4)),
    (tbp.NN, (2552, 2312, 1032), (256, 128, 1, 1)), (tbp.NT, (2104, 2064, 1056), (256, 128, 1, 1)), (tbp.NN, (920, 1400, 4904), (256, 128, 1, 5)),
    (tbp.NT, (936, 1328, 4744), (256, 128, 1, 4)),
    (tbp.NN, (1448, 5768, 144), (192, 192, 1, 1)), (tbp.NT, (1064, 7520, 160), (192, 192, 1, 1)), (tbp.NN, (1296, 976, 4952), (192, 192, 1, 6)),
    (tbp.NT, (520, 2200, 4128), (192, 192, 1, 6)),
    (tbp.NN, (1736, 4904, 368), (256, 192, 1, 1)), (tbp.NT, (1936, 4440, 368), (256, 192, 1, 1)), (tbp.NN, (984, 2056, 4472), (256, 192, 1, 5)),
    (tbp.NT, (1240, 3224, 3232), (256, 192, 1, 3)),
    (tbp.NN, (2576, 4712, 384), (256, 256, 1, 1)), (tbp.NT, (2192, 5400, 392), (256, 256, 1, 1)), (tbp.NN, (2120, 2000, 4144), (256, 256, 1, 3)),
    (tbp.NT, (2224, 1936, 4168), (256, 256, 1, 3))]


def to_dev(a: np.ndarray, dtype: str) -> torch.Tensor:
    """float32 array that is exactly representable in `dtype` -> device tensor of that storage type."""
    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32))
    return t.to(DEV, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32).contiguous()


def to_np(t: torch.Tensor) -> np.ndarray:
    return t.detach().to("cpu", dtype=torch.float64).numpy()


def max_rel(got, ref) -> float:
    """max |got - ref| / max |ref|   (the max-norm relative error used for every tolerance here)."""
    ref = np.asarray(ref, np.float64)
    got = np.asarray(got, np.float64)
    assert got.shape == ref.shape, (got.shape, ref.shape)
    if ref.size == 0:
        return 0.0
    assert np.all(np.isfinite(got)), "non-finite values in the GPU result"
    return float(np.max(np.abs(got - ref)) / max(np.max(np.abs(ref)), 1e-300))


def stage_tolerance(dtype: str) -> float:
    # stated tolerance of the benchmark definition: 1e-4 in fp32 mode, 2e-2 for bf16 against fp64
    return 2e-2 if dtype == "bf16" else 1e-4


def make_gpu_stage(shape: si.StageShape, params: dict, **kw):
    dev_params = {k: [to_dev(w, shape.dtype) for w in v] for k, v in params.items() if v}
    return tbp.Stage(tbp.config_from_shape(shape, **kw), dev_params, DEV)


def run_oracle(shape, params, xs, dys, concat=False):
    st = oracle.OracleStage(shape, params)
    outs = [st.forward(m, xs[m]) for m in range(len(xs))]
    dxs = [st.backward_p1(m, dys[m]) for m in range(len(xs))]
    st.backward_p2(range(len(xs)), concat=concat)
    return outs, dxs, st.grads()


def compare_stage(shape, gpu_outs, gpu_dxs, gpu_grads, outs, dxs, grads, tol, label=""):
    worst = {}
    for m in range(len(outs)):
        worst[f"x_out[{m}]"] = max_rel(to_np(gpu_outs[m]), outs[m])
        worst[f"dx[{m}]"] = max_rel(to_np(gpu_dxs[m]), dxs[m])
    for k, lst in gpu_grads.items():
        for l, g in enumerate(lst):
            worst[f"d{k}[{l}]"] = max_rel(to_np(g), grads[k][l])
    bad = {k: v for k, v in worst.items() if not v <= tol}
    top = sorted(worst.items(), key=lambda kv: -kv[1])[:4]
    print(f"[parity {label}] worst={max(worst.values()):.3e} tol={tol:g} over {len(worst)} tensors; largest: "
          + ", ".join(f"{k}={v:.2e}" for k, v in top), flush=True)
    assert not bad, bad
    return worst
