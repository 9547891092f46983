"""decode_vq: the fp32-precision decode kernel for the calls outside the table
kernels' head counts and layouts, against the fp64 oracle.

Lengths at the edges of its 16-token tiles and 64-token rounds, contiguous
capacities and pages that are no multiple of 16, several counts of query heads
per KV head, windows, sinks, bands that the window cuts, the formats, and
values far outside fp16's range (each head's q' and the scalar arm's weights
carry a power of two of their own).

Tolerance: q', the probabilities and every sum carry fp32 rounding, so a logit
z (|z| < 16 here) errs by a few |z| 2^-24 and a probability by as much
relative: 16 x 4 x 2^-24 = 4e-6; 1e-5 of the row norm."""

import numpy as np
import pytest
import torch

import synth
from helpers import assert_outputs_close, pool_offsets
from oracle import attention as oatt
from oracle import codec as ocodec
from oracle import fp8 as ofp8

pytestmark = pytest.mark.gpu
TOL32 = 1e-5


@pytest.fixture(scope="module")
def nk():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2608_04074_amd as nk
    nk._native.lib()
    return nk


def dev(x, dtype):
    return torch.as_tensor(np.ascontiguousarray(x)).to(dtype).cuda()


def bits(x):
    return torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).cuda()


EDGES = [0, 1, 15, 16, 17, 63, 64, 65, 600, 1201]
CASES = [
    # D, query heads per KV head, block size (None: contiguous), format flags, window, band, sinks
    (128, 8, None, "", 0, None, False),
    (128, 5, 16, "", 0, None, True),
    (128, 7, 32, "fp8", 100, None, True),
    (128, 8, None, "ks sq", 0, (64, 256), True),
    (128, 6, 16, "ks fp8 sq bf16", 90, (5, 70), True),
    (128, 1, 24, "ks", 0, (3, 0), False),
    (128, 4, 8, "sq", 33, None, True),
    (64, 8, None, "ks sq", 0, (0, 17), True),
    (64, 3, 5, "fp8 bf16", 0, (20, 40), False),
    (128, 8, None, "wide ks sq", 0, None, False),
    (64, 8, None, "wide", 0, None, False),
]


@pytest.mark.parametrize("D,gqa,bs,fmt,window,band,use_sink", CASES)
def test_against_oracle(nk, D, gqa, bs, fmt, window, band, use_sink):
    fmt = fmt.split()
    ks, sq, fp8, bf16, wide = (f in fmt for f in ("ks", "sq", "fp8", "bf16", "wide"))
    H = 2
    wl = synth.get_workload("qwen3_8b" if D == 128 else "gptoss_pair").scaled(num_kv_heads=H, num_q_heads=H * gqa)
    lens = np.array(EDGES, np.int32)
    B, cap, L = len(lens), 1201, D // 4
    rng = np.random.default_rng(D + gqa)
    arr = dict(synth.bench_params(wl))
    if wide:  # the same logits from q' of 2^60 and scales of 2^-60 (2^14 and smaller codewords without scales)
        arr["t_k_inv_t"] = arr["t_k_inv_t"] * np.float32(2.0 ** (60 if ks else 14))
        if not ks:
            arr["cb_k"], arr["cb_v"] = ((arr[k].astype(np.float32) * 2.0 ** -14).astype(np.float16) for k in ("cb_k", "cb_v"))
    if fp8:
        for k in ("cb_k", "cb_v"):
            arr[k] = ofp8.e4m3_bits(ofp8.snap_e4m3(arr[k].astype(np.float64)))
    params = dict(arr)
    if fp8:
        for k in ("cb_k", "cb_v"):
            params[k] = ofp8.e4m3_value(arr[k])
    if bf16:
        for k in ("t_k", "t_k_inv_t", "t_v"):
            params[k] = synth.round_to_bf16(arr[k])
    if sq:
        arr["cb_v"] = None
    P = nk.NovaKVParams.from_arrays(arr, key_scale=ks, sq_values=sq, bf16_transforms=bf16)
    bps = 1 if bs is None else -(-cap // bs)
    rows = cap if bs is None else bs
    table = None if bs is None else rng.permutation(B * bps).astype(np.int32).reshape(B, bps)
    lay = nk.CacheLayout.contiguous(cap) if bs is None else nk.CacheLayout(bs, bps, dev(table, torch.int32))
    shape = (B * bps, H, rows)
    ck, cv = (rng.integers(0, 256, shape + (L,), dtype=np.uint8) for _ in range(2))
    kscale = ocodec.bf16_bits(np.exp(0.3 * rng.standard_normal(shape)) * (2.0 ** -60 if wide else 1.0))
    vs = np.exp(0.3 * rng.standard_normal(shape)) * (2.0 ** 100 if wide else 1.0)
    vsq = np.stack([ocodec.bf16_bits(vs), ocodec.bf16_bits(vs * (-1.5 + 0.2 * rng.standard_normal(shape)))], -1)
    q = rng.standard_normal((B, H * gqa, D)).astype(np.float32)
    sinks = rng.standard_normal(H * gqa).astype(np.float32) if use_sink else None
    bnd = None
    if band:
        nb = sum(band)
        hb = ocodec.bf16_bits(rng.standard_normal((2, B, H, nb, D)))
        bnd = nk.Band(*band, bits(hb[0]), bits(hb[1]))
        slot = lambda p: p if p < band[0] else band[0] + p % band[1]  # noqa: E731
    print(f"[gpu-case] decode_vq D={D} gqa={gqa} block={bs} {fmt} window={window} band={band}", flush=True)
    out = nk.decode_attn(P, lay, dev(q, torch.float32), dev(ck, torch.uint8), dev(cv, torch.uint8),
                         dev(lens, torch.int32), cap, window=window,
                         sinks=dev(sinks, torch.float32) if use_sink else None,
                         k_scales=bits(kscale) if ks else None, v_sq=bits(vsq) if sq else None, band=bnd).cpu().numpy()
    ref = np.zeros(out.shape)
    for b in range(B):
        n = int(lens[b])
        for kv in range(H):
            off = pool_offsets(b, kv, np.arange(n), hkv=H, groups=1, block_size=rows, blocks_per_seq=bps, table=table)
            hp = oatt.head_params({k: v for k, v in params.items() if v is not None}, kv)
            ex = None
            if band:
                m = oatt.band_mask(n, *band)
                rows_k, rows_v = (np.zeros((n, D)) for _ in range(2))
                for p in np.flatnonzero(m):
                    rows_k[p], rows_v[p] = (ocodec.bf16_value(hb[i, b, kv, slot(p)]) for i in (0, 1))
                ex = (*band, rows_k, rows_v)
            s2 = vsq.reshape(-1, 2)[off]
            hs = slice(kv * gqa, (kv + 1) * gqa)
            ref[b, hs] = oatt.decode_rows(q[b, hs].astype(np.float64), ck.reshape(-1, L)[off], cv.reshape(-1, L)[off], hp,
                                          1 / np.sqrt(D), window, None if sinks is None else sinks[hs],
                                          scales_k=ocodec.bf16_value(kscale.reshape(-1)[off]) if ks else None, band=ex,
                                          sq_v=(s2[:, 0], s2[:, 1]) if sq else None)
    assert not out[0].any()
    assert_outputs_close(out.reshape(-1, D), ref.reshape(-1, D), tol=TOL32, what=f"decode_vq D={D} gqa={gqa} {bs} {fmt}")


@pytest.mark.parametrize("n", [7001, 20011, 60001])
def test_combine_of_many_splits(nk, n):
    """One KV head over up to 40 splits, which the combine reads eight at a
    time; the second sequence leaves all but the first of them empty."""
    B, H, gqa, D, L = 2, 1, 8, 128, 32
    wl = synth.get_workload("qwen3_8b").scaled(num_kv_heads=H, num_q_heads=gqa)
    arr = dict(synth.bench_params(wl))
    P = nk.NovaKVParams.from_arrays(arr)
    rng = np.random.default_rng(n)
    codes = rng.integers(0, 256, (2, B, n, L), dtype=np.uint8)
    q = rng.standard_normal((B, gqa, D)).astype(np.float32)
    lens = np.array([n, 129], np.int32)
    print(f"[gpu-case] decode_vq many splits n={n}", flush=True)
    out = nk.decode_attn(P, nk.CacheLayout.contiguous(n), dev(q, torch.float32), dev(codes[0][:, None], torch.uint8),
                         dev(codes[1][:, None], torch.uint8), dev(lens, torch.int32), n).cpu().numpy()
    hp = oatt.head_params(arr, 0)
    ref = np.stack([oatt.decode_rows(q[b].astype(np.float64), codes[0, b, :m], codes[1, b, :m], hp, 1 / np.sqrt(D), 0, None)
                    for b, m in enumerate(lens)])
    assert_outputs_close(out.reshape(-1, D), ref.reshape(-1, D), tol=TOL32, what=f"decode_vq of {n} tokens")


@pytest.mark.parametrize("D,cap", [(64, 20011), (64, 20016), (128, 20011)])
def test_one_workspace_for_several_shapes(nk, D, cap):
    """A workspace zero-filled once serves calls of any batch: the partials that
    one sequence's splits leave lie past the arrival counters of 300."""
    L, B = D // 4, 300
    wl = synth.get_workload("qwen3_8b" if D == 128 else "gptoss_pair").scaled(num_kv_heads=1, num_q_heads=1)
    P = nk.NovaKVParams.from_arrays(dict(synth.bench_params(wl)))
    lay = nk.CacheLayout.contiguous(cap)
    gen = torch.Generator(device="cuda").manual_seed(D)
    ck, cv = (torch.randint(0, 256, (B, 1, cap, L), generator=gen, device="cuda", dtype=torch.uint8) for _ in range(2))
    q = torch.randn((B, 1, D), generator=gen, device="cuda")
    lens = torch.full((B,), cap, dtype=torch.int32, device="cuda")
    print(f"[gpu-case] one workspace for batches of 1 and {B}, D={D} cap={cap}", flush=True)
    ref = nk.decode_attn(P, lay, q, ck, cv, lens, cap)
    ws = torch.zeros(max(nk.decode_workspace_bytes(P, b, 1, cap) for b in (1, B)), dtype=torch.uint8, device="cuda")
    for n in (1, B, 1, B):
        out = torch.full((n, 1, D), float("nan"), device="cuda")
        nk.decode_attn(P, lay, q[:n].contiguous(), ck[:n], cv[:n], lens[:n].contiguous(), cap, out=out, workspace=ws)
        assert_outputs_close(out.cpu().numpy().reshape(-1, D), ref[:n].cpu().numpy().reshape(-1, D).astype(np.float64),
                             tol=TOL32 if cap % 16 else 2e-3, what=f"shared workspace D={D} cap={cap} batch {n}")
