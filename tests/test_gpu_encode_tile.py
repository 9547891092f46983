"""encode_tile: the tiled append encoder against the fp64 oracle.

Its search scores codewords with split fp16 operands, takes the best block of
eight, and falls back to fp64 where the runner-up is within the error bound, so
its codes are the fp64 argmin, the smallest index among equal distances.  Cases:
tiles that straddle sequences, a tile of a few tokens, both launch shapes (one
group per wave, and all four), both head sizes; codebooks far larger and far
smaller than the coefficients (the group's and the token's scales), a repeated
codeword (a tie), and a codeword that is not finite; and what leaves many tokens
of a group undecided, which the group is then scored once more for: codebooks of
mostly repeated codewords (zeros of both signs among them), groups of little
variance, tokens far larger than the codebook."""

import numpy as np
import pytest
import torch

import synth
from helpers import compare_codes
from oracle import attention as oatt
from oracle import codec as ocodec
from oracle import fp8 as ofp8

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nk():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2608_04074_amd as nk
    nk._native.lib()
    return nk


def dev(x, dtype):
    return torch.as_tensor(np.ascontiguousarray(x)).to(dtype).cuda()


@pytest.mark.parametrize("D,B,n_new,H", [(128, 3, 5, 2), (128, 7, 13, 2), (64, 5, 33, 2), (64, 2, 129, 1),
                                         (128, 2, 1055, 4), (64, 3, 1400, 4)])
@pytest.mark.parametrize("kind", ["plain", "ties", "scales", "repeated", "little variance", "large tokens"])
def test_codes(nk, D, B, n_new, H, kind):
    wl = synth.get_workload("qwen3_8b" if D == 128 else "gptoss_pair").scaled(num_kv_heads=H, num_q_heads=H)
    params = dict(synth.bench_params(wl))
    for k in ("cb_k", "cb_v"):
        c = params[k].astype(np.float32).copy()
        if kind == "ties":
            c[:, :, 100] = c[:, :, 7]
        elif kind == "scales":
            L = c.shape[1]
            c *= (2.0 ** np.array([12, -12, 3, -3, 0, 6, -20])[np.arange(L) % 7])[None, :, None, None].astype(np.float32)
            c[:, L - 1, 9, 2] = np.inf
        elif kind == "repeated":
            c[:, :, 40:] = c[:, :, 39 - np.arange(40, 256) % 37]
            c[:, 1::4] *= 0.0  # zeros of both signs only
        elif kind == "little variance":
            c[:, ::2] *= 2.0 ** -10
        params[k] = c.astype(np.float16)
    P = nk.NovaKVParams.from_arrays(params)
    rng = np.random.default_rng(n_new)
    cap = n_new + 11
    start = rng.integers(0, 12, B).astype(np.int32)
    kk, vv = (torch.as_tensor(rng.standard_normal((B, n_new, H, D))).to(torch.bfloat16) for _ in range(2))
    if kind == "scales":  # tokens much larger and smaller than their neighbours
        s = torch.as_tensor(2.0 ** rng.integers(-6, 7, (B, n_new, 1, 1)))
        kk, vv = (kk.double() * s).to(torch.bfloat16), (vv.double() * s).to(torch.bfloat16)
    elif kind == "large tokens":
        kk, vv = (x * 512 for x in (kk, vv))
    elif kind == "little variance":  # as little in the same groups' coefficients
        w = torch.ones(D // 4, 4, dtype=torch.float64)
        w[::2] = 2.0 ** -10
        t = [torch.as_tensor(np.asarray(params[n], np.float64)) for n in ("t_k_inv_t", "t_v", "kbar")]
        kk, vv = (torch.matmul((x.double() * w.reshape(-1))[..., None, :], m.transpose(1, 2).contiguous())[..., 0, :]
                  for x, m in ((kk, t[0]), (vv, t[1])))
        kk, vv = (kk + t[2]).float(), vv.float()
    pk = torch.zeros((B, H, cap, D // 4), dtype=torch.uint8, device="cuda")
    pv = torch.zeros_like(pk)
    print(f"[gpu-case] encode_tile D={D} B={B} n_new={n_new} H={H} {kind}", flush=True)
    nk.encode(P, nk.CacheLayout.contiguous(cap), kk.cuda(), vv.cuda(), dev(start, torch.int32), pk, pv)
    hk, hv = pk.cpu().numpy(), pv.cpu().numpy()
    kd, vd = kk.double().numpy(), vv.double().numpy()
    with np.errstate(all="ignore"):
        for b in range(B):
            s0 = int(start[b])
            assert not hk[b, :, :s0].any() and not hk[b, :, s0 + n_new:].any()
            for kv in range(H):
                ck, gk, cv, gv = ocodec.encode_tokens(kd[b, :, kv], vd[b, :, kv], oatt.head_params(params, kv))
                got_k, got_v = hk[b, kv, s0:s0 + n_new], hv[b, kv, s0:s0 + n_new]
                compare_codes(got_k, ck, gk, f"encode_tile D={D} {kind} b{b} kv{kv} K")
                compare_codes(got_v, cv, gv, f"encode_tile D={D} {kind} b{b} kv{kv} V")
                if kind == "repeated":  # never one that repeats another
                    assert not (got_k[:, 0::4] >= 40).any() and not got_k[:, 1::4].any() and not got_v[:, 1::4].any()
                if kind == "ties":
                    assert not (got_k == 100).any() and not (got_v == 100).any()


@pytest.mark.parametrize("D,B,n_new,fmt", [(128, 3, 2735, ""), (128, 3, 5466, "key_scale"), (64, 3, 5465, ""),
                                           (64, 5, 3300, "fp8 bf16"), (128, 1, 8192, "f32")])
def test_two_tiles_per_workgroup(nk, D, B, n_new, fmt):
    """Launches large enough for workgroups of two tiles (the last of them with
    an empty, a partial or a full second tile) store what calls of one sequence
    or of a quarter of it store, which take a workgroup per tile; the oracle on
    some tokens of them."""
    H, L = 8, D // 4
    wl = synth.get_workload("qwen3_8b" if D == 128 else "gptoss_pair").scaled(num_kv_heads=H, num_q_heads=H)
    params = dict(synth.bench_params(wl))
    arr, ks = dict(params), "key_scale" in fmt
    if "fp8" in fmt:
        for k in ("cb_k", "cb_v"):
            arr[k] = ofp8.e4m3_bits(ofp8.snap_e4m3(arr[k].astype(np.float64)))
            params[k] = ofp8.e4m3_value(arr[k])
    if "bf16" in fmt:
        for k in ("t_k", "t_k_inv_t", "t_v"):
            params[k] = synth.round_to_bf16(arr[k])
    P = nk.NovaKVParams.from_arrays(arr, key_scale=ks, bf16_transforms="bf16" in fmt)
    rng = np.random.default_rng(n_new)
    cap = n_new + 11
    start = rng.integers(0, 12, B).astype(np.int32)
    dt = torch.float32 if "f32" in fmt else torch.bfloat16
    kk, vv = (torch.as_tensor(rng.standard_normal((B, n_new, H, D))).to(dt).cuda() for _ in range(2))
    sp = dev(start, torch.int32)

    def pools():
        p = [torch.zeros((B, H, cap, L), dtype=torch.uint8, device="cuda") for _ in range(2)]
        return p + ([torch.zeros((B, H, cap), dtype=torch.bfloat16, device="cuda")] if ks else [])

    def encode(p, b0, b1, t0, t1):
        p = [x[b0:b1] for x in p]
        nk.encode(P, nk.CacheLayout.contiguous(cap), kk[b0:b1, t0:t1].contiguous(), vv[b0:b1, t0:t1].contiguous(),
                  (sp[b0:b1] + t0).contiguous(), p[0], p[1], **(dict(k_scales=p[2]) if ks else {}))

    print(f"[gpu-case] encode_fast, two tiles per workgroup, D={D} B={B} n_new={n_new} {fmt}", flush=True)
    whole, parts = pools(), pools()
    encode(whole, 0, B, 0, n_new)
    for b in range(B):
        for t0 in range(0, n_new, 2735):
            encode(parts, b, b + 1, t0, min(n_new, t0 + 2735))
    for w, p in zip(whole, parts):
        assert torch.equal(w, p)
    tail = slice(n_new - 30, n_new)
    s0, kd, vd = int(start[B - 1]), kk[B - 1, tail].double().cpu().numpy(), vv[B - 1, tail].double().cpu().numpy()
    for kv in (0, H - 1):
        ck, gk, cv, gv = ocodec.encode_tokens(kd[:, kv], vd[:, kv], oatt.head_params(params, kv))
        rows = slice(s0 + n_new - 30, s0 + n_new)
        if not ks:
            compare_codes(whole[0][B - 1, kv, rows].cpu().numpy(), ck, gk, f"encode_fast pairs D={D} kv{kv} K")
        compare_codes(whole[1][B - 1, kv, rows].cpu().numpy(), cv, gv, f"encode_fast pairs D={D} kv{kv} V")


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D,B,n_new,H,ks,sq", [(128, 3, 13, 2, False, False), (64, 3, 40, 2, True, True),
                                               (128, 2, 1055, 4, False, False), (64, 3, 1400, 4, True, False),
                                               (128, 3, 2735, 8, False, False), (64, 3, 5465, 8, False, True)])
def test_inputs_at_any_address(nk, dtype, D, B, n_new, H, ks, sq):
    """Keys and values that start one element into a buffer are loaded element by
    element; the codes, scales and band rows are those of the same inputs at an
    aligned address (which vectors load)."""
    wl = synth.get_workload("qwen3_8b" if D == 128 else "gptoss_pair").scaled(num_kv_heads=H, num_q_heads=H)
    arr = dict(synth.bench_params(wl))
    if sq:
        arr["cb_v"] = None
    P = nk.NovaKVParams.from_arrays(arr, key_scale=ks, sq_values=sq)
    gen = torch.Generator(device="cuda").manual_seed(n_new)
    k, v = (torch.randn((B, n_new, H, D), generator=gen, device="cuda").to(dtype) for _ in range(2))
    start = torch.zeros(B, dtype=torch.int32, device="cuda")

    def shifted(x):
        y = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")[1:].view(x.shape)
        y.copy_(x)
        assert y.data_ptr() % 8 != 0
        return y

    def encode(kk, vv):
        shape = (B, H, n_new)
        out = {"k": torch.zeros(shape + (D // 4,), dtype=torch.uint8, device="cuda"),
               "v": torch.zeros(shape + (D // 4,), dtype=torch.uint8, device="cuda"),
               "ks": torch.zeros(shape, dtype=torch.bfloat16, device="cuda") if ks else None,
               "sq": torch.zeros(shape + (2,), dtype=torch.bfloat16, device="cuda") if sq else None}
        band = nk.Band(3, 20, *(torch.zeros((B, H, 23, D), dtype=torch.bfloat16, device="cuda") for _ in range(2)))
        nk.encode(P, nk.CacheLayout.contiguous(n_new), kk, vv, start, out["k"], out["v"], k_scales=out["ks"],
                  v_sq=out["sq"], band=band)
        return [*(x for x in out.values() if x is not None), band.k, band.v]

    print(f"[gpu-case] encode from an odd address D={D} B={B} n_new={n_new} {dtype} ks={ks} sq={sq}", flush=True)
    for x, y in zip(encode(k, v), encode(shifted(k), shifted(v))):
        assert torch.equal(x, y)
