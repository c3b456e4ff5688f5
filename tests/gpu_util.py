"""Helpers for the GPU tests: move seeded inputs to the device with padded
rows whose padding holds NaN (so any use of padding shows up), and bring
outputs back as float64."""
import re

import numpy as np
import pytest
import torch

NAN_BF16 = 0x7FC0


def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def dev_mat(storage, dtype, device, pad_value=float("nan"), align=None):
    """Device tensor [R][C] with a leading dimension rounded up to the
    library's alignment and NaN in the padding columns."""
    storage = np.ascontiguousarray(storage)
    R, C = storage.shape
    if align is None:
        align = 8 if dtype == "bf16" else 4
    ld = max((C + align - 1) // align * align, align)
    if dtype == "bf16":
        full = np.full((R, ld), NAN_BF16, dtype=np.uint16)
        full[:, :C] = storage
        t = torch.from_numpy(full.view(np.int16)).view(torch.bfloat16)
    else:
        full = np.full((R, ld), pad_value, dtype=np.float32)
        full[:, :C] = storage
        t = torch.from_numpy(full)
    return t.to(device)[:, :C]


def out_mat(R, C, dtype, device, fill=float("nan")):
    """Output tensor [R][C] (padded leading dimension) prefilled with `fill`,
    so unwritten entries and writes into padding are visible."""
    align = 8 if dtype == "bf16" else 4
    ld = max((C + align - 1) // align * align, align)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    return torch.full((R, ld), fill, dtype=tdt, device=device)[:, :C]


def host64(t):
    return t.float().cpu().numpy().astype(np.float64)


def padding(t):
    """The padding columns [C, ld) of a padded 2-D view, as a host array."""
    R, C = t.shape
    ld = t.stride(0)
    base = t.as_strided((R, ld), (ld, 1))
    return base[:, C:].float().cpu().numpy()


TILES = {0: "256x256", 3: "128x128", 4: "256x256", 5: "256x256", 6: "128x192",
         7: "256x192", 8: "192x192", 9: "256x160"}


def plans(capfd, call):
    """(call(), the plans of the bfloat16 products it ran): one dict each, with the
    sizes R, Cc, D, the kind of kernel, the tile's name (tiled) or index (small
    tiles), the depth ranges (splits), whether two are combined inside the kernel
    (pair), and rows1, tile2, ... of a second launch by rows; of an MX-FP8 product
    (out_mx: the projection) the small-tile configuration (small, or -1) and the
    projection's tile otherwise (0: 256 x 256, 1: 128 x 128, 2: 128 x 192)."""
    capfd.readouterr()
    out = call()
    got = []
    for mx, line in re.findall(r"^espace (mx )?plan (.*)$", capfd.readouterr().err, re.M):
        p = {k: int(v) for k, v in re.findall(r"(\w+)=(-?\d+)", line)}
        if mx:
            got.append(p)
            continue
        p["kind"] = {0: "tiled", 1: "small", 3: "gemv", 4: "stream"}[p["kind"]]
        if p["kind"] == "tiled":
            p["tile"], p["tile2"] = TILES[p["tile"]], TILES[p["tile2"]]
        got.append(p)
    return out, got
