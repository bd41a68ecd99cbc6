"""GPU parity of the quantiser variants (Sec. 3.1, App. D) with the fp64
oracle: the (b+1)-bit alphabet, scales per column group and per column, the
MSE scale search, and a block-diagonal output factor."""
import numpy as np
import pytest

import workloads
from gpu_util import block_diag, check_against_oracle, gpu_run, gpu_run_antidiag, log

pytestmark = pytest.mark.gpu


def _variant(m, n, seed, bits, alphabet, group, cols):
    """A random problem with the quantiser variant: group scales are max-abs
    per (row, group) over the largest code, column factors in [0.5, 1.5]."""
    p = workloads.make_random(m, n, seed=seed, bits=bits)
    r = np.random.Generator(np.random.PCG64(np.random.SeedSequence([7200, m, n, seed])))
    hi = (1 << (bits - 1)) - 1
    W = p["W"]
    if group:
        G = -(-n // group)
        sc = np.zeros((m, G), np.float32)
        for g in range(G):
            sc[:, g] = np.max(np.abs(W[:, g * group:(g + 1) * group]), axis=1) / np.float32(hi)
        p["scale"] = sc.astype(np.float32)
        p["group_size"] = group
    p["alphabet"] = alphabet
    if cols:
        p["col_scale"] = r.uniform(0.5, 1.5, n).astype(np.float32)
    return p


@pytest.mark.parametrize("alphabet,group,cols", [("asym", 0, False), ("sym", 32, False),
                                                  ("sym", 0, True), ("asym", 48, True)])
@pytest.mark.parametrize("m,n,bits", [(70, 90, 3), (33, 129, 2), (130, 67, 4)])
def test_quantiser_variant_parity(oracle_mod, alphabet, group, cols, m, n, bits):
    p = _variant(m, n, 300 + m + n, bits, alphabet, group, cols)
    log(f"case quant {alphabet} g={group} cols={cols} m={m} n={n} bits={bits}")
    codes, V, pre = gpu_run(p)
    check_against_oracle(p, codes, V, pre, oracle_mod, label=f"q-{alphabet}-{group}-{cols}")


def test_quantiser_variant_knear0_and_antidiag(oracle_mod):
    """Every (source, target) pair through the node kernels (KNEAR = 0), and
    Alg. 3's per-diagonal rounding, with the most general quantiser."""
    p = _variant(100, 97, 17, 3, "asym", 16, True)
    log("case quant knear=0")
    codes, V, pre = gpu_run(p, k=0)
    check_against_oracle(p, codes, V, pre, oracle_mod, label="q-knear0")
    log("case quant antidiag")
    codes, V, pre = gpu_run_antidiag(p)
    check_against_oracle(p, codes, V, pre, oracle_mod, label="q-antidiag")


def test_unit_column_factors_are_bitwise_per_row(oracle_mod):
    """Column factors of 1 and groups as wide as the matrix take the general
    path but must reproduce the per-row solve bit for bit (s * 1 = s)."""
    p = workloads.make_random(150, 140, seed=23, bits=4)
    log("case quant unit factors")
    c0, v0, x0 = gpu_run(p)
    q = dict(p, col_scale=np.ones(140, np.float32))
    c1, v1, x1 = gpu_run(q)
    g = dict(p, scale=p["scale"].reshape(150, 1).copy(), group_size=140)
    c2, v2, x2 = gpu_run(g)
    for c, v, x in ((c1, v1, x1), (c2, v2, x2)):
        assert np.array_equal(c, c0) and np.array_equal(v.view(np.uint32), v0.view(np.uint32))
        assert np.array_equal(np.isnan(x), np.isnan(x0)) and np.array_equal(x[~np.isnan(x)],
                                                                           x0[~np.isnan(x0)])


@pytest.mark.parametrize("bits,alphabet,group", [(3, "sym", 0), (4, "asym", 0), (2, "asym", 0),
                                                 (3, "sym", 32), (4, "sym", 100)])
def test_mse_scales_parity(oracle_mod, bits, alphabet, group):
    """The same scale as the oracle's search (identical fp32 decisions); a
    different pick is accepted only where two candidates' fp64 errors agree to
    1e-12 (summation order)."""
    import torch
    import paper_2608_06291_amd as pk
    r = np.random.Generator(np.random.PCG64(np.random.SeedSequence([7300, bits, group])))
    m, n = 97, 301
    W = (r.standard_t(4, (m, n)) * 0.02).astype(np.float32)
    W[5] = 0.0
    W[7, :] = 0.01
    log(f"case mse scales bits={bits} {alphabet} g={group}")
    got = pk.mse_scales(torch.from_numpy(W).to("cuda:0"), bits, alphabet, group_size=group)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    ref, err = oracle_mod.mse_scales(W, bits, alphabet, group_size=group)
    assert got.shape == ref.shape
    diff = np.argwhere(got != ref)
    log(f"[mse] {len(diff)} of {got.size} scales differ")
    for idx in diff:
        idx = tuple(int(v) for v in idx)
        seg = W if group == 0 else W[:, idx[1] * group:(idx[1] + 1) * group]
        cand = oracle_mod.mse_scale_candidates(seg, bits, alphabet)[idx[0]]
        hit = np.flatnonzero(cand == got[idx])
        assert hit.size, (idx, "not a candidate scale")
        e = err[idx]
        assert abs(e[hit[0]] - e.min()) <= 1e-12 * e.min(), idx
    # the scales drive a solve: per-row MSE scales through the solver
    if group == 0:
        p = workloads.make_random(m, 64, seed=5, bits=bits)
        p["W"] = W[:, :64].copy()
        p["alphabet"] = alphabet
        p["scale"], _ = oracle_mod.mse_scales(p["W"], bits, alphabet)
        codes, V, pre = gpu_run(p)
        check_against_oracle(p, codes, V, pre, oracle_mod, label="mse-solve")


@pytest.mark.parametrize("exp", [0, -123, -140, 110, 124])
@pytest.mark.parametrize("alphabet", ["sym", "asym"])
def test_mse_scales_boundaries(oracle_mod, exp, alphabet):
    """Entries on and one ulp beside the rounding boundaries (k + 1/2) s, for
    scales in the middle of fp32's range, subnormal ones and ones whose
    reciprocal is subnormal: the same picks as the oracle's IEEE divisions."""
    import torch
    import paper_2608_06291_amd as pk
    log(f"case mse boundaries exp={exp} {alphabet}")
    bits = 8
    k = np.arange(-128, 128, dtype=np.float64)
    half = ((k + 0.5) * 2.0 ** -4).astype(np.float32)
    rows = [np.concatenate([half, np.nextafter(half, np.float32(np.inf)),
                            np.nextafter(half, np.float32(-np.inf)), [np.float32(t)]])
            for t in (127 * 2.0 ** -4, 9.0, 11.3)]
    W = np.ldexp(np.array(rows, np.float32), exp).astype(np.float32)
    got = pk.mse_scales(torch.from_numpy(W).to("cuda:0"), bits, alphabet).cpu().numpy()
    ref, err = oracle_mod.mse_scales(W, bits, alphabet)
    for i in range(len(rows)):
        if got[i] != ref[i]:   # another pick only where the fp64 sums agree
            cand = oracle_mod.mse_scale_candidates(W, bits, alphabet)[i]
            hit = np.flatnonzero(cand == got[i])
            assert hit.size and abs(err[i][hit[0]] - err[i].min()) <= 1e-12 * err[i].min()


@pytest.mark.parametrize("nheads,hb,n", [(4, 32, 80), (3, 48, 70), (8, 16, 33)])
def test_block_diagonal_B_parity(oracle_mod, nheads, hb, n):
    """B = blockdiag of per-head Grams (App. D): parity with the oracle on the
    assembled matrix, and the factor is exactly block-diagonal."""
    import torch
    import paper_2608_06291_amd as pk
    p = workloads.make_random(nheads * hb, n, seed=nheads * 100 + hb)
    r = np.random.Generator(np.random.PCG64(np.random.SeedSequence([7400, nheads, hb])))
    blocks = []
    for h in range(nheads):
        X = workloads.ar1_samples(4 * hb, hb, 0.3 + 0.1 * (h % 3), r).astype(np.float64)
        blocks.append((X.T @ X / (4 * hb)).astype(np.float32))
    p["B_blocks"] = np.stack(blocks)
    p["B"] = None
    log(f"case blockdiag heads={nheads} hb={hb} n={n}")
    codes, V, pre = gpu_run(p)
    check_against_oracle(p, codes, V, pre, oracle_mod, label=f"bd{nheads}x{hb}")
    A = torch.from_numpy(p["A"]).to("cuda:0")
    f = pk.factor_blockdiag(A, torch.from_numpy(p["B_blocks"]).to("cuda:0"), p["damp"])
    LB = f.export("B").cpu().numpy()
    f.close()
    off = LB.copy()
    for h in range(nheads):
        off[h * hb:(h + 1) * hb, h * hb:(h + 1) * hb] = 0
    assert np.count_nonzero(off) == 0
    ref = oracle_mod.normalized_factor(block_diag(p["B_blocks"]), p["damp"])
    assert np.max(np.abs(LB - ref)) < 1e-5 * max(1.0, np.max(np.abs(ref)))
