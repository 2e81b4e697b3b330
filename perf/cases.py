"""The work that users of this library have it do, as measurable cases.

A case is one call of a public entry point, or the few calls of one decoder layer, on synthetic matrices shaped like the
ones the repository's configurations and tests use.  Matrices are built as the offline side builds them: Gaussian weights,
min-max quantised per row and group at the width of their tile, packed by sfmp_pack, resident on the GPU.

Fields of a case
  call    "gemm"  one sfmp_gemm call
          "batch" independent projections of one input sharing a launch (sfmp_gemv_batched / sfmp_gemm_batched)
          "layer" the seven projections of a decoder layer in the four calls a layer can use:
                  q|k|v, o, gate|up, down
  M       activation rows: 1 = one decoded token, 2..16 = a small decode batch, above = a prompt
  K, N    input and output features (N2, N3: further projections of a "batch"; for "layer" K is the hidden size, N the
          feed-forward size and N2 the width of k and v)
  mix     share of tiles per bit-width: "234" thirds of 2/3/4 bits, "23" and "34" halves, "2344" a quarter of 2 and
          3 bits and a half of 4 bits, "2", "3", "4" one width
  group, fmt       columns per (scale, zero) pair and their storage type
  block_n, block_k tiles per bit-allocation block, rows and columns
  outliers         1 % of the activation columns are 20 times larger
  col_perm, row_perm   whether the call reorders activations and un-permutes outputs
"""
import math

import numpy as np
import torch

import paper_2602_01027_amd as S
import sfmp_workloads as W

DEVICE = "cuda:0"

MIXES = {"234": {2: 1 / 3, 3: 1 / 3, 4: 1 / 3}, "23": {2: 0.5, 3: 0.5}, "34": {3: 0.5, 4: 0.5},
         "2344": {2: 0.25, 3: 0.25, 4: 0.5}, "2": {2: 1.0}, "3": {3: 1.0}, "4": {4: 1.0}}

# the largest matrix and the largest prompt of the repository's configurations
MAX_WEIGHTS = 28672 * 8192
MAX_DIM = 28672
MAX_M = 2048


def _case(call, M, K, N, **more):
    c = dict(call=call, M=M, K=K, N=N, N2=0, N3=0, mix="234", group=128, fmt="fp16", block_n=1, block_k=1,
             outliers=False, col_perm=True, row_perm=True)
    c.update(more)
    return c


def listed():
    named = [
        # the smallest configuration: a call that is all launch and latency
        ("gemv_512", _case("gemm", 1, 512, 512)),
        # one decoded token through an 8B-shaped layer, average 3.0 bits: the repository's headline workload
        ("decode_layer_8b", _case("layer", 1, 4096, 14336, N2=1024)),
        # one decoded token, q|k|v in the paper's own parameter format: (512, 256) blocks, group 256, bf16 parameters
        ("decode_qkv_bf16_g256", _case("batch", 1, 4096, 4096, N2=1024, N3=1024, group=256, fmt="bf16", block_n=4,
                                       block_k=2)),
        # one decoded token through the largest matrix of a 70B-shaped layer, average 3.25 bits
        ("decode_70b_gate", _case("gemm", 1, 8192, 28672, mix="2344")),
        # four and sixteen sequences decoded together, fractional 2.5 bits, activations with outlier columns
        ("batch4_layer_8b", _case("layer", 4, 4096, 14336, N2=1024, mix="23", outliers=True)),
        ("batch16_layer_8b", _case("layer", 16, 4096, 14336, N2=1024, mix="23", outliers=True)),
        # eight sequences through the longest reduction
        ("batch8_70b_down", _case("gemm", 8, 28672, 8192, mix="2344")),
        # a short prompt, or 64 sequences at once
        ("prompt64_8b_gate", _case("gemm", 64, 4096, 14336, mix="23", outliers=True)),
        # a short prompt of odd length through a long reduction, two parameter pairs per tile column
        ("prompt200_8b_down_g64", _case("gemm", 200, 14336, 4096, group=64)),
        # a prompt of odd length through a square projection
        ("prompt777_8b_q", _case("gemm", 777, 4096, 4096, mix="34", outliers=True)),
        # full prefill blocks: the wide 8B matrix, and the largest matrix left in reordered row order
        ("prefill2048_8b_gate", _case("gemm", 2048, 4096, 14336, mix="34", outliers=True)),
        ("prefill2048_70b_down", _case("gemm", 2048, 28672, 8192, mix="34", outliers=True, row_perm=False)),
    ]
    return [dict(c, name=n) for n, c in named]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _features(rng, most, unit=128, least=512):
    """A feature count: a multiple of `unit`, spread over the logarithm of the range, odd multiples among them."""
    return max(least, min(most, _log_int(rng, least, most) // unit * unit)) // unit * unit


def draw(rng):
    """Another case of the same ranges: M from 1 to 2048, features from 512 to 28672, every option of the entry points."""
    call = rng.choice(("gemm", "gemm", "gemm", "batch"))
    regime = rng.choice(("token", "batch", "short", "prompt")) if call == "gemm" else rng.choice(("token", "batch"))
    lo, hi = {"token": (1, 1), "batch": (2, 16), "short": (17, 256), "prompt": (257, MAX_M)}[regime]
    M = _log_int(rng, lo, hi)
    group = rng.choice((128, 128, 128, 64, 256, 512))
    unit = max(128, group)
    K = _features(rng, MAX_DIM, unit, max(512, unit))
    most_n = min(MAX_DIM, MAX_WEIGHTS // K)
    c = _case(call, M, K, 0, mix=rng.choice(tuple(MIXES)), group=group, fmt=rng.choice(("fp16", "fp16", "bf16")),
              block_k=unit // 128, outliers=rng.random() < 0.5, col_perm=rng.random() < 0.85,
              row_perm=rng.random() < 0.8)
    if call == "batch":
        c["N"] = _features(rng, min(most_n, 14336), least=256)
        c["N2"] = _features(rng, max(256, min(most_n - c["N"], 14336)), least=256)
        c["N3"] = rng.choice((0, _features(rng, 4096, least=256)))
    else:
        c["N"] = _features(rng, most_n)
    return c


def _projections(case):
    """(K, N) of every projection, and how they are grouped into calls."""
    K, N, N2, N3 = case["K"], case["N"], case["N2"], case["N3"]
    if case["call"] == "gemm":
        return [(K, N)], [[0]]
    if case["call"] == "batch":
        shapes = [(K, n) for n in (N, N2, N3) if n]
        return shapes, [list(range(len(shapes)))]
    return [(K, K), (K, N2), (K, N2), (K, K), (K, N), (K, N), (N, K)], [[0, 1, 2], [3], [4, 5], [6]]


def _bitmap(case, K, N, rng):
    bn, bk = case["block_n"], case["block_k"]
    if (N // 128) % bn:
        bn = 1
    return W.block_bitmap(N // 128, K // 128, MIXES[case["mix"]], rng, bn, bk)


def _quantised(case, K, N, bitmap, gen):
    """Codes [N, K] (host) and stored scales / zeros [K/group, N] of a Gaussian matrix, min-max quantised on the GPU."""
    g = case["group"]
    store = torch.float16 if case["fmt"] == "fp16" else torch.bfloat16
    codes = torch.empty((N, K), dtype=torch.uint8, device=DEVICE)
    scales = torch.empty((K // g, N), dtype=store, device=DEVICE)
    zeros = torch.empty_like(scales)
    levels_of = (2.0 ** torch.from_numpy(bitmap.astype(np.float32)) - 1.0).to(DEVICE)  # [N/128, K/128]
    std = 0.02 if K * N < 64 * 2 ** 20 else 0.015
    rows = max(1, (1 << 26) // (K * 128)) * 128  # a bounded piece of the matrix at a time
    for r0 in range(0, N, rows):
        r1 = min(N, r0 + rows)
        w = torch.empty((r1 - r0, K), dtype=torch.float32, device=DEVICE).normal_(0.0, std, generator=gen)
        w = w.view(r1 - r0, K // g, g)
        lv = levels_of[r0 // 128:r1 // 128]
        lv = lv[:, ::g // 128] if g >= 128 else lv.repeat_interleave(128 // g, dim=1)
        lv = lv.repeat_interleave(128, dim=0)  # [rows, K/g]
        lo, hi = w.amin(dim=2), w.amax(dim=2)
        s, z = ((hi - lo) / lv).to(store), lo.to(store)
        q = ((w - z.float()[:, :, None]) / s.float()[:, :, None]).round_().clamp_(min=0.0)
        codes[r0:r1] = torch.minimum(q, lv[:, :, None]).to(torch.uint8).view(r1 - r0, K)
        scales[:, r0:r1], zeros[:, r0:r1] = s.t(), z.t()
    return codes.cpu().numpy(), scales, zeros


def _matrix(case, K, N, gen, rng):
    bitmap = _bitmap(case, K, N, rng)
    codes, scales, zeros = _quantised(case, K, N, bitmap, gen)
    layout, s2, s3, s4, index = S.sfmp_pack(codes, bitmap)
    S.sfmp_layout_set_quant(layout, case["group"], case["fmt"])

    def up(a):
        return torch.from_numpy(a).to(DEVICE)

    packed = S.DevicePacked(layout, up(s2), up(s3), up(s4), up(index), scales.view(torch.float16),
                            zeros.view(torch.float16), up(bitmap))
    col = up(W.make_perm(K, rng)) if case["col_perm"] else None
    row = up(W.make_perm(N, rng)) if case["row_perm"] else None
    return packed, col, row


def _activations(case, K, gen):
    x = torch.empty((case["M"], K), dtype=torch.float32, device=DEVICE).normal_(generator=gen)
    if case["outliers"]:
        x[:, torch.randperm(K, device=DEVICE, generator=gen)[:K // 100]] *= 20.0
    return x.to(torch.float16)


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    rng = np.random.default_rng([seed, 0x5F3])
    M = case["M"]
    shapes, calls = _projections(case)
    matrices = [_matrix(case, K, N, gen, rng) for K, N in shapes]
    outputs = [torch.empty((M, N), dtype=torch.float16, device=DEVICE) for _, N in shapes]
    state = dict(call=case["call"], M=M, outputs=outputs, calls=[])
    for members in calls:
        X = _activations(case, shapes[members[0]][0], gen)  # the projections of a call read the same activations
        problems = [(X, matrices[i][1], matrices[i][0], matrices[i][2], outputs[i]) for i in members]
        if case["call"] == "gemm":
            nbytes = S.sfmp_gemm_workspace(problems[0][2].layout, M)
        else:
            nbytes = S.sfmp_gemm_batched_workspace(problems, M)
        state["calls"].append((problems, torch.empty(nbytes, dtype=torch.uint8, device=DEVICE)))
    return state


def run(state):
    for problems, workspace in state["calls"]:
        if state["call"] == "gemm":
            X, col, p, row, Y = problems[0]
            S.sfmp_gemm(X, col, p.layout, p.s2, p.s3, p.s4, p.index, p.scales, p.zeros, p.bitmap, row, Y, workspace)
        elif state["M"] == 1:
            S.sfmp_gemv_batched(problems)
        else:
            S.sfmp_gemm_batched(problems, state["M"], workspace)
    return state["outputs"]


def work(case):
    shapes, calls = _projections(case)
    M, nbytes, flops = case["M"], 0, 0
    for K, N in shapes:
        bitmap = _bitmap(case, K, N, np.random.default_rng(0))  # (the number of tiles of each width is fixed by the mix)
        nbytes += W.algorithmic_bytes(N, K, M, bitmap, col_perm=case["col_perm"], row_perm=case["row_perm"],
                                      index_words=bitmap.size, group=case["group"])
        flops += 2 * M * N * K
    for members in calls:  # activations that several projections share are read once
        nbytes -= 2 * M * shapes[members[0]][0] * (len(members) - 1)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # fp16 outputs of fp32 sums, with the dequantised weight rounded once to fp16 on the matrix-core path: against the
    # same product in 64 bits the 2-norm is off by 2.0e-4 to 2.8e-4 and the largest element by up to 1.5e-3 of the
    # larger of its value and the root mean square
    return {"rel": 1.2e-3, "max": 6e-3}
