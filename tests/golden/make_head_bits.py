"""Writes head_bits.json: the latents that the diffusion head samples, bit for
bit.

    python tests/golden/make_head_bits.py

The head's results are a fixed function of its inputs: row statistics, the
output product and the sampler sum in one stated order (a lane's columns in
ascending order, then a fixed tree over the lanes), and the products in one
order of k.  The file was written by the library when every stage was a kernel
of its own with one wave per row, and is not rewritten when kernels are fused
or rows are spread over more waves: those must keep the bits.

Needs the GPU and the built library of the tree in the working folder.
"""
from __future__ import annotations

import json
import os
import sys

import numpy as np

OUT = os.path.join(os.path.dirname(os.path.abspath(__file__)), "head_bits.json")

# width, depth, token_dim, tokens, sampling steps: the widths of the models
# (1024, 1280, 1536), widths that fill neither a wave nor a lane group, more
# than 2048, the widest; tokens of few components, of more than 16 and of 64;
# enough rows that the products take other tiles
CASES = [(1024, 2, 16, 5, 6), (1280, 2, 16, 5, 6), (1536, 2, 16, 5, 6), (128, 2, 16, 300, 5), (192, 2, 3, 7, 6),
         (320, 1, 64, 3, 5), (640, 1, 15, 9, 5), (1792, 1, 16, 4, 5), (2112, 1, 24, 3, 5), (2560, 1, 16, 3, 5),
         (4096, 1, 16, 3, 4), (4096, 1, 33, 2, 4)]


def name(case) -> str:
    return "width %d, depth %d, token_dim %d, %d tokens, %d steps" % tuple(case)


def sample(case) -> np.ndarray:
    """The latents of a case's (at most eight) first tokens, float32."""
    import torch

    from paper_2503_12450_amd import binding as B
    from paper_2503_12450_amd.device import to_device, upload_head
    from paper_2503_12450_amd.workload import HeadDims, head_weights, normal_rows

    width, depth, T, R, steps = case
    hd = HeadDims(width=width, depth=depth, cond_dim=64, token_dim=T, steps=steps, train_steps=10 * steps,
                  freq_dim=64, max_rows=R)
    head = B.MarHead(hd, upload_head(head_weights(hd, seed=51), hd.dtype))
    yc, yu = (to_device(normal_rows((R, hd.cond_dim), seed=s, std=2.0), "f32") for s in (52, 53))
    idx = torch.arange(R, dtype=torch.int32, device="cuda")
    x0 = to_device(normal_rows((R, T), seed=54), "f32")
    xi = to_device(normal_rows((steps, R, T), seed=55), "f32")
    out = torch.empty((R, T), device="cuda")
    head.sample(yc, yu, idx, idx, x0, xi, 3.0, out)
    torch.cuda.synchronize()
    return out.cpu().numpy()[:8]


def main() -> None:
    data = {"_about": "float32 bit patterns (hex) of the sampled latents, per case of tests/golden/make_head_bits.py"}
    for case in CASES:
        x = sample(case)
        assert np.all(np.isfinite(x))
        data[name(case)] = ["".join("%08x" % v for v in row) for row in x.view(np.uint32)]
        print(name(case), flush=True)
    with open(OUT, "w") as f:
        json.dump(data, f, indent=1)
        f.write("\n")


if __name__ == "__main__":
    sys.path.insert(0, os.getcwd())
    main()
