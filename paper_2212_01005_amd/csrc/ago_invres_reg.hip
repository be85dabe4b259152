// Plans and launches of the register-resident pointwise -> depthwise -> pointwise kernel (ago_invres_reg.hpp).
#include "ago_invres_reg.hpp"
#include <algorithm>

namespace ago {

namespace {
constexpr size_t kLdsMax = 160 * 1024;
// channels per workgroup when the expanded channels are split over workgroups (0: not)
constexpr int kSplits[4] = {0, 64, 128, 256};
constexpr int kParts[4] = {1, 2, 4, 8};
constexpr int kWaves[2] = {4, 8};
}  // namespace

int invres_reg_num_cfgs() { return 2 * 4 * 2 * 4 * 2; }

// Fill p and q for configuration cfg = ropt + 2 (parts option + 4 (waves option + 2 (split option + 4 chunked))).  False: does not apply.
bool invres_reg_plan_cfg(InvresRegPlan& q, int cfg, int N, int H, int W, int Cin, int Cexp, int Cout, int stride, int ksize, bool bf16) {
    InvresRegParams& p = q.p;
    p = InvresRegParams{};
    const int ropt = cfg & 1, nwc = kParts[(cfg >> 1) & 3], nw = kWaves[(cfg >> 3) & 1], split = kSplits[(cfg >> 4) & 3];
    const int es = bf16 ? 2 : 4, kg = bf16 ? 32 : 16, pad = (ksize - 1) / 2;
    if (nwc > nw) return false;
    const int cot = (Cout + 15) / 16;
    int nco = 0;
    for (int v : kRegNco)
        if (nco == 0 && v >= cot) nco = v;
    if (nco == 0) nco = kRegNco[3];
    int nk = (Cin + kg - 1) / kg, xr = 0;
    if (bf16) xr = nk <= 5 ? nk : 0;
    else xr = nk <= 2 ? 2 : nk <= 4 ? 4 : 0;
    const int R = kRegR[stride - 1][ropt];
    // parts of a unit would each load the same fragments: beyond two steps the waves of four or more parts share them in LDS
    if (nwc >= 4 && nk > 2) xr = 0;
    if (xr && reg_need(bf16, stride, ksize, R, xr, nco) > 256) xr = 0;
    if (xr) nk = xr;
    if (R == 4 && (nco > 4 || xr == 0)) return false;
    p.N = N; p.H = H; p.W = W; p.Cin = Cin; p.Cexp = Cexp; p.Cout = Cout;
    p.OH = (H - 1) / stride + 1; p.OW = (W - 1) / stride + 1;
    p.rows = R; p.nk = nk;
    const int lh = stride == 1 ? pad : 1, vx = 16 - lh - (stride == 1 ? pad : ksize == 5 ? 1 : 0);
    // two row blocks side by side need the columns beyond the map as separators: the widest reach of a tap
    p.segs = p.OW <= 8 - (stride == 1 ? pad : 1) ? 2 : 1;
    p.strips = p.segs == 2 ? 1 : (p.OW + vx - 1) / vx;
    p.yblocks = (p.OH + R - 1) / R;
    p.rowblocks = N * p.yblocks;
    p.units = (p.rowblocks + p.segs - 1) / p.segs * p.strips;
    // 32-bit offsets, and divisions by multiplication exact below 2^32
    if ((long)N * H * W * Cin * es >= (1L << 31) || (long)N * p.OH * p.OW * Cout * 4 >= (1L << 31) || (long)p.units * p.strips >= (1L << 32) ||
        (long)p.rowblocks * p.yblocks >= (1L << 32) || (long)Cexp * std::max(Cin, Cout) * es >= (1L << 31))
        return false;
    p.x_bytes = (unsigned)((long)N * H * W * Cin * es);
    p.out_elems = (unsigned)((long)N * p.OH * p.OW * Cout);
    p.inv_strips = 0xffffffffu / p.strips + 1;
    p.inv_yblocks = 0xffffffffu / p.yblocks + 1;
    p.nwc_log = (cfg >> 1) & 3; p.nwu = nw / nwc;
    q.cogroups = (cot + nco - 1) / nco;
    p.csplit = split ? split : Cexp;
    if (split && split >= Cexp) return false;
    const bool chunked = cfg >= 64;
    if (chunked && (!split || ropt)) return false;
    p.cspan = chunked ? Cexp : p.csplit;
    p.nsplit = (Cexp + p.cspan - 1) / p.cspan;
    const int tiles = p.csplit / 16;                                         // of expanded channels, divided among the parts
    if (tiles < nwc) return false;
    const int rows = (R - 1) * stride + ksize, cow = std::min(nco * 16, Cout);
    const long xbytes = xr ? 0 : (long)p.nwu * rows * stride * nk * 1024;
    p.p1 = p.csplit * es;
    p.p2 = cow * es;
    auto kb = [](long v) { return (v + 1023) / 1024; };
    p.n1 = (int)kb((long)nk * kg * p.p1); p.n2 = (int)kb((long)p.csplit * p.p2);
    // the last load of each may run past its rows; a projection tile reads 16 NCO output channels from a row on
    const long w1_bytes = p.n1 * 1024L, w2_bytes = std::max<long>(p.n2 * 1024L, (long)(p.csplit - 1) * p.p2 + nco * 16 * es), tw_bytes = (long)tiles * (2 + ksize * ksize) * 64;
    const long bytes = (w1_bytes + w2_bytes + 15) / 16 * 16 + tw_bytes + xbytes;
    if (bytes > (long)kLdsMax) return false;
    p.off_w2 = (int)w1_bytes;
    p.off_wd = (int)((w1_bytes + w2_bytes + 15) / 16 * 16);
    p.off_x = p.off_wd + (int)tw_bytes;
    p.q2 = cow * es / 16;
    p.inv2 = 0xffffffffu / p.q2 + 1;                                         // several groups of output channels: q2 > 1
    p.q1_log = 0;
    while ((16 << p.q1_log) < p.p1) ++p.q1_log;                              // split: csplit is a power of two
    q.xr = xr; q.nco = nco; q.ropt = ropt; q.threads = nw * 64;
    // workgroups along the units: all of them, or as many as stay resident when the weights are staged once
    const long need = ((long)p.units + p.nwu - 1) / p.nwu;
    long red = nwc > 1 ? (long)p.nwu * nwc * R * nco * 1024 : 0;
    auto finish = [&](long groups) {
        q.groups = (int)groups;
        const bool alias = groups >= need;                                   // the weights are dead by then
        p.off_red = alias ? 0 : (int)bytes;
        q.smem = (size_t)(alias ? std::max(bytes, red) : bytes + red);
    };
    finish(need);
    // (two of exactly half the LDS were not seen side by side)
    const long resident = std::max<long>(1, std::min<long>((long)((kLdsMax - 1) / q.smem), 4 * reg_waves(bf16, stride, ksize, R, xr, nco) / nw));
    const long slots = 256 * resident / (q.cogroups * p.nsplit) > 0 ? 256 * resident / (q.cogroups * p.nsplit) : 1;
    if (need > slots) {
        const long rounds = (need + slots - 1) / slots;
        finish((need + rounds - 1) / rounds);                                // balanced rounds
    }
    if (q.smem > kLdsMax) return false;
    const long wgs = (long)q.groups * q.cogroups;
    if (wgs >= (1L << 31) || p.nsplit > 65535) return false;

    // Time model (us), fitted to about 2500 timed launches of 84 shapes (5 % rms): staging; fragments; the units a wave
    // walks, each its share of the channel tiles, bound by the wave's own chain of instructions or, with several waves
    // per SIMD, by what they issue together; the sum over parts; the sum over workgroups (a second launch).
    const double frags = rows * stride, mfma = (bf16 ? 16.0 : 128.0) * (frags * nk + R * nco);
    const double valu = 2.1 * frags + (ksize == 3 ? 18.3 : 16.3) * ksize * ksize * R + 5.0;
    const double lds = nk * (bf16 ? 2 : 4) + ksize * ksize + nco * (bf16 ? 1 : 4) + (xr ? 0.0 : frags * nk);
    const long wgs_all = wgs * p.nsplit, per_round = 256 * resident;
    const double wgs_cu = (double)std::min<long>((wgs_all + 255) / 256, resident), rounds = (double)((wgs_all + per_round - 1) / per_round);
    const double per_simd = std::max(1.0, wgs_cu * nw / 4.0), ppw = (tiles + nwc - 1) / nwc;
    const double alone = valu + (bf16 ? 2.2 : 1.15) * mfma + 20.0 * lds, shared = valu + (bf16 ? 1.95 * mfma + 5.8 * lds : 1.2 * mfma);
    const double walk = ppw * std::max(alone, per_simd * shared), stage_n = p.n1 + p.n2;
    double stage = (34.0 / nw + 14.3 * wgs_cu) * stage_n + 124.0 * ((tiles + 16 * nw - 1) / (16 * nw)) * ksize * ksize;
    double unit = walk + frags * nk * (bf16 ? 2 : 1) * (xr ? 125.0 : 120.0 / nwc) + 104.0 * R * nco * (nwc == 1);
    if (nwc > 1) unit += 1085.0 + 33.0 * R * nco * (1 + nwc);
    if (chunked) {
        const double chunks = (p.cspan + p.csplit - 1) / p.csplit;
        unit += (chunks - 1) * walk + chunks * (stage + 700.0);
        stage = 0.0;
    }
    double us = 2.24 + rounds * (stage + (double)((need + q.groups - 1) / q.groups) * unit) / 2400.0;
    if (p.nsplit > 1) us += 1.78 + 0.02 * Cin + 0.84 * (p.nsplit + 1) * N * p.OH * p.OW * Cout * 1e-6;
    q.us = us;
    return true;
}

size_t invres_reg_split_bytes(const InvresRegPlan& q) {
    const InvresRegParams& p = q.p;
    return p.nsplit > 1 ? (size_t)p.nsplit * p.N * p.OH * p.OW * p.Cout * sizeof(float) : 0;
}

hipError_t invres_reg_launch(const InvresRegPlan& q, int stride, int ksize, bool bf16, hipStream_t s) {
    const unsigned grid = (unsigned)q.groups;
    auto* fn = bf16 ? (stride == 1 ? (ksize == 3 ? invres_reg_b13 : invres_reg_b15) : (ksize == 3 ? invres_reg_b23 : invres_reg_b25))
                    : (stride == 1 ? (ksize == 3 ? invres_reg_f13 : invres_reg_f15) : (ksize == 3 ? invres_reg_f23 : invres_reg_f25));
    return fn(q.ropt, q.xr, q.nco, q.p, grid, (unsigned)q.threads, q.smem, s);
}

}  // namespace ago
