"""Shared test plumbing: tensor <-> numpy views, block-wise oracle evaluation, the head's division of its products."""
import functools
import os
import subprocess
import tempfile

import numpy as np
import torch

from oracle import grpo_oracle as orc


def logits_to_numpy(t):
    """torch [n, V] float32 or bfloat16 (any device, row-strided) -> numpy the oracle accepts."""
    t = t.detach().cpu()
    if t.dtype == torch.bfloat16:
        return t.contiguous().view(torch.int16).numpy().view(np.uint16)
    return t.contiguous().numpy()


def grads_to_f64(t):
    return t.detach().cpu().to(torch.float64).numpy()


def oracle_logprobs_blocked(batch, block_rows=4096, progress=None):
    """Oracle log-probs for every row of a (possibly device-resident) batch, streaming
    the logits to the host in row blocks so that they never sit there as a whole."""
    N = batch["n_tokens"]
    lp = np.zeros(N, dtype=np.float64)
    tokens = batch["tokens"].cpu().numpy()
    mask = batch["mask"].cpu().numpy()
    for r0 in range(0, N, block_rows):
        r1 = min(N, r0 + block_rows)
        if not mask[r0:r1].any():
            continue
        z = logits_to_numpy(batch["logits"][r0:r1])
        lp[r0:r1] = orc.logprobs(z, tokens[r0:r1], mask[r0:r1], temperature=batch["temperature"])
        if progress:
            progress(r1)
    return lp


def sample_rows_by_class(coeff, mask, rng, per_class):
    """Row indices covering every row class: masked, zero-coefficient, live."""
    masked = np.flatnonzero(mask == 0)
    zero_c = np.flatnonzero((mask == 1) & (coeff == 0))
    live = np.flatnonzero((mask == 1) & (coeff != 0))
    pick = []
    for cls in (masked, zero_c, live):
        if len(cls):
            pick.append(rng.choice(cls, size=min(per_class, len(cls)), replace=False))
    return np.sort(np.concatenate(pick)) if pick else np.zeros(0, dtype=np.int64)


@functools.lru_cache(maxsize=None)
def _lm_plan_program():
    folder = tempfile.mkdtemp(prefix="lm_plan")
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_07291_amd", "csrc")
    src, exe = os.path.join(folder, "plan.cpp"), os.path.join(folder, "plan")
    with open(src, "w") as f:
        f.write("""#include <cstdio>
#include <cstdlib>
#include "lm_plan.hpp"
int main(int, char **a)
{
    const LmPlan p = lm_plan(atoi(a[1]), atoi(a[2]), atoi(a[3]), atoi(a[4]), atoi(a[5]), atoi(a[6]));
    printf("%d %d %d %d %d %d %d\\n", p.full, p.rest, p.s2, p.halves, p.thin, p.t2, p.pairs);
}
""")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", csrc, "-o", exe, src], check=True)
    return exe


def lm_plan(rows, cols, depth, split_blocks=0):
    """How lm_gemm_nt divides a product of rows x cols over a contraction of depth on this GPU (csrc/lm_plan.hpp, taken
    by the host compiler); split_blocks: the partial blocks there is room for, where the contraction may be cut."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    args = [rows, (cols + 255) // 256, (depth + 63) // 64, 1 if split_blocks else 0, split_blocks, cus]
    out = subprocess.run([_lm_plan_program()] + [str(a) for a in args], check=True, capture_output=True, text=True).stdout
    return dict(zip(("full", "rest", "s2", "halves", "thin", "t2", "pairs"), map(int, out.split())))
