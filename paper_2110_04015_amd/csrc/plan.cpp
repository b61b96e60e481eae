// Host-side planning of the HBM layout: landmark order, 64-slot tiles, chunks,
// and the deterministic camera reductions.  Integer work only; every floating
// point step runs in the HIP kernels.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <utility>

#include "ba_internal.h"

namespace ba {

// Subset s = floor(np / N) holds poses [s*p, s*(p+1)) for p < N-1; the last
// subset holds the rest (Sec. 3.2, "Optimized implementation").
void partition_groups(int np, int N, int32_t *group) {
    int s = np / N;
    for (int c = 0; c < np; ++c) {
        int g = c / s;
        group[c] = g < N - 1 ? g : N - 1;
    }
}

static void counting_csr(const int32_t *key, int64_t m, int nk, std::vector<int64_t> &ptr,
                         std::vector<int64_t> &idx) {
    ptr.assign((size_t)nk + 1, 0);
    idx.resize((size_t)m);
    for (int64_t o = 0; o < m; ++o) ptr[(size_t)key[o] + 1]++;
    for (int k = 0; k < nk; ++k) ptr[k + 1] += ptr[k];
    std::vector<int64_t> fill(ptr.begin(), ptr.end() - 1);
    for (int64_t o = 0; o < m; ++o) idx[(size_t)fill[(size_t)key[o]]++] = o;
}

// Chunks of consecutive tiles with at most max_slots distinct cameras; scam: camera of every
// slot.  C may be P's own (its meta words hold the landmark indices already).
static void make_chunks(const HostPlan &P, const std::vector<int32_t> &scam, int max_slots, int max_tiles, int shares,
                        HostChunks &C) {
    const int np = P.np;
    const int64_t tiles = P.n_tiles;
    // with a number of chunks to make, they take equal shares of the tiles in turn (whole
    // tiles: floor or ceiling): with every chunk of the same length some lengths (43, 55 and
    // their doubles among those tried) cost the product 10 % or more, and a ceiling for all
    // leaves the last round short
    if (shares > 0) max_tiles = (int)std::min<int64_t>(4096, std::max<int64_t>(1, (tiles + shares - 1) / shares));
    C.max_tiles = max_tiles;
    std::vector<int32_t> stamp((size_t)np, -1), slot_of((size_t)np, 0);
    std::vector<int64_t> tstamp((size_t)np, -1);
    C.chunk_tile.clear();
    C.chunk_part.clear();
    C.chunk_seg.clear();
    C.part_cam.clear();
    int64_t chunk = -1;
    int slots = 0, ntiles_in = 0, room = max_tiles;
    for (int64_t t = 0; t < tiles; ++t) {
        int fresh = 0;   // cameras of tile t not yet in the current chunk
        for (int q = 0; q < kTile; ++q) {
            const int c = scam[(size_t)(t * kTile + q)];
            if (c < 0) break;
            if (stamp[(size_t)c] != chunk && tstamp[(size_t)c] != t) {
                tstamp[(size_t)c] = t;
                ++fresh;
            }
        }
        if (chunk < 0 || slots + fresh > max_slots || ntiles_in >= room || P.tile_seg[(size_t)t] != C.chunk_seg.back()) {
            ++chunk;
            slots = 0;
            ntiles_in = 0;
            if (shares > 0) {
                const int64_t share = (chunk + 1) * tiles / shares - chunk * tiles / shares;
                room = (int)std::min<int64_t>(max_tiles, std::max<int64_t>(1, share));
            }
            C.chunk_tile.push_back((int32_t)t);
            C.chunk_part.push_back((int32_t)C.part_cam.size());
            C.chunk_seg.push_back(P.tile_seg[(size_t)t]);
        }
        for (int q = 0; q < kTile; ++q) {
            const size_t sidx = (size_t)(t * kTile + q);
            const int c = scam[sidx];
            if (c < 0) break;
            if (stamp[(size_t)c] != chunk) {
                stamp[(size_t)c] = (int32_t)chunk;
                slot_of[(size_t)c] = slots++;
                C.part_cam.push_back(c);
            }
            C.meta[sidx] = meta_pack((uint32_t)slot_of[(size_t)c], P.meta[sidx] >> 16);
        }
        ++ntiles_in;
    }
    C.n_chunks = (int)chunk + 1;
    C.chunk_tile.push_back((int32_t)tiles);
    C.chunk_part.push_back((int32_t)C.part_cam.size());
    C.n_part = (int64_t)C.part_cam.size();
    C.max_used_slots = 1;
    for (int ch = 0; ch < C.n_chunks; ++ch)
        C.max_used_slots = std::max(C.max_used_slots, C.chunk_part[(size_t)ch + 1] - C.chunk_part[(size_t)ch]);
    // camera-major CSR over partial rows (ascending row order = fixed summation order)
    std::vector<int64_t> ptr, idx;
    counting_csr(C.part_cam.data(), C.n_part, np, ptr, idx);
    C.cam_part_ptr.resize((size_t)np + 1);
    for (int c = 0; c <= np; ++c) C.cam_part_ptr[(size_t)c] = (int32_t)ptr[(size_t)c];
    C.cam_part_idx.resize((size_t)C.n_part);
    for (int64_t i = 0; i < C.n_part; ++i) C.cam_part_idx[(size_t)i] = (int32_t)idx[(size_t)i];
    // a chunk writes its partial row straight into the camera-major position
    C.part_dst.resize((size_t)C.n_part);
    for (int64_t j = 0; j < C.n_part; ++j) C.part_dst[(size_t)C.cam_part_idx[(size_t)j]] = (int32_t)j;
}

void build_chunks(const HostPlan &P, int max_slots, int max_tiles, int shares, HostChunks &C) {
    std::vector<int32_t> scam((size_t)P.n_tiles * kTile, -1);
    for (int ch = 0; ch < P.n_chunks; ++ch) {
        const int32_t *cams = P.part_cam.data() + P.chunk_part[(size_t)ch];
        for (int64_t sl = (int64_t)P.chunk_tile[(size_t)ch] * kTile; sl < (int64_t)P.chunk_tile[(size_t)ch + 1] * kTile; ++sl)
            if (P.meta[(size_t)sl] != kPad) scam[(size_t)sl] = cams[P.meta[(size_t)sl] & 0xFFFFu];
    }
    C.meta.assign(P.meta.size(), kPad);
    make_chunks(P, scam, max_slots, max_tiles, shares, C);
}

ba_status build_plan(int np, int nl, int64_t m, const int32_t *cam, const int32_t *lm,
                     int max_slots, int max_tiles, HostPlan &P, std::string &err, const int32_t *cam_seg,
                     int target_chunks, int max_tiles_multi, int target_multi, int shares) {
    char buf[256];
    P = HostPlan();
    P.np = np;
    P.nl = nl;
    P.m = m;
    P.max_slots = max_slots;
    P.max_tiles = max_tiles > 0 ? max_tiles : 16;
    P.max_tiles_multi = max_tiles_multi > 0 ? max_tiles_multi : max_tiles > 0 ? max_tiles : 16;
    for (int64_t o = 0; o < m; ++o) {
        if (cam[o] < 0 || cam[o] >= np || lm[o] < 0 || lm[o] >= nl) {
            snprintf(buf, sizeof buf, "observation %lld has camera %d / landmark %d out of range",
                     (long long)o, cam[o], lm[o]);
            err = buf;
            return BA_ERR_INVALID_ARG;
        }
    }
    P.obs_cam.assign(cam, cam + m);
    std::vector<int64_t> lptr, lobs;
    counting_csr(lm, m, nl, lptr, lobs);

    // per landmark: observations sorted by camera, duplicate check, min camera
    std::vector<int32_t> minc((size_t)nl, 0), lcam((size_t)m);   // lcam: cameras of lobs
    for (int l = 0; l < nl; ++l) {
        int64_t a = lptr[l], b = lptr[l + 1];
        int64_t c = b - a;
        if (c > kTile) {
            snprintf(buf, sizeof buf, "landmark %d has %lld observations; at most %d are supported", l,
                     (long long)c, kTile);
            err = buf;
            return BA_ERR_UNSUPPORTED;
        }
        bool sorted = true;
        for (int64_t q = a; q < b; ++q) {
            lcam[(size_t)q] = cam[lobs[(size_t)q]];
            sorted = sorted && (q == a || lcam[(size_t)q] > lcam[(size_t)q - 1]);
        }
        if (!sorted) {
            std::pair<int32_t, int64_t> by_cam[kTile];
            for (int64_t q = a; q < b; ++q) by_cam[q - a] = {lcam[(size_t)q], lobs[(size_t)q]};
            std::sort(by_cam, by_cam + c);
            for (int64_t q = a; q < b; ++q) {
                lcam[(size_t)q] = by_cam[q - a].first;
                lobs[(size_t)q] = by_cam[q - a].second;
            }
        }
        for (int64_t q = a + 1; q < b; ++q) {
            if (lcam[(size_t)q] == lcam[(size_t)q - 1]) {
                snprintf(buf, sizeof buf, "camera %d observes landmark %d twice", lcam[(size_t)q], l);
                err = buf;
                return BA_ERR_INVALID_ARG;
            }
        }
        if (c == 0) {
            snprintf(buf, sizeof buf, "landmark %d has no observation: V_lambda is singular", l);
            err = buf;
            return BA_ERR_NOT_SPD;
        }
        minc[l] = lcam[(size_t)a];
        if (cam_seg && cam_seg[lcam[(size_t)b - 1]] != cam_seg[minc[l]]) {
            snprintf(buf, sizeof buf, "landmark %d is observed by cameras of two problems of the batch", l);
            err = buf;
            return BA_ERR_INVALID_ARG;
        }
    }
    if (cam_seg) {
        for (int c = 1; c < np; ++c)
            if (cam_seg[c] < cam_seg[c - 1]) {
                err = "the problems of a batch must hold consecutive cameras";
                return BA_ERR_INVALID_ARG;
            }
        P.cam_seg.assign(cam_seg, cam_seg + np);
    }
    auto seg_of_lmk = [&](int l) { return cam_seg ? cam_seg[minc[(size_t)l]] : 0; };
    // landmark storage order: by smallest observing camera (stable counting sort), so
    // that consecutive landmarks share cameras on banded problems
    {
        std::vector<int64_t> cnt((size_t)np + 2, 0);
        for (int l = 0; l < nl; ++l) cnt[(size_t)minc[l] + 1]++;
        for (int k = 0; k <= np; ++k) cnt[k + 1] += cnt[k];
        P.lmk_order.resize((size_t)nl);
        for (int l = 0; l < nl; ++l) P.lmk_order[(size_t)cnt[(size_t)minc[l]]++] = l;
    }
    std::vector<int32_t> scam;   // camera of every slot
    // tiles: landmarks never straddle a tile boundary.  Tiles are filled from a
    // window of the next kWindow landmarks of the sorted order: a landmark that
    // does not fit the current tile waits while later ones fill the gap, and the
    // oldest waiting landmark always opens the next tile.  The storage order of
    // the landmarks becomes their placement order.
    {
        constexpr int kWindow = 48;
        std::vector<int32_t> sorted = P.lmk_order;
        std::vector<int32_t> pending;
        pending.reserve(kWindow);
        P.lmk_order.clear();
        P.lmk_order.reserve((size_t)nl);
        P.lmk_first_slot.resize((size_t)nl);
        P.lmk_count.resize((size_t)nl);
        P.slot_obs.clear();
        P.meta.clear();
        P.slot_obs.reserve((size_t)m + (size_t)m / 16 + kTile);
        P.meta.reserve((size_t)m + (size_t)m / 16 + kTile);
        scam.reserve((size_t)m + (size_t)m / 16 + kTile);
        P.tile_lmk_base.clear();
        size_t next = 0;
        int64_t t = 0;
        while (next < (size_t)nl || !pending.empty()) {
            while (pending.size() < (size_t)kWindow && next < (size_t)nl) pending.push_back(sorted[next++]);
            P.tile_lmk_base.push_back((int32_t)P.lmk_order.size());
            P.slot_obs.resize((size_t)(t + 1) * kTile, -1);
            P.meta.resize((size_t)(t + 1) * kTile, kPad);
            scam.resize((size_t)(t + 1) * kTile, -1);
            // a tile holds landmarks of one problem: that of the oldest waiting landmark
            const int tseg = seg_of_lmk(pending[0]);
            P.tile_seg.push_back(tseg);
            int used = 0, ll = 0;
            size_t keep = 0;
            for (size_t i = 0; i < pending.size(); ++i) {
                int l = pending[i];
                int c = (int)(lptr[l + 1] - lptr[l]);
                if (used + c > kTile || seg_of_lmk(l) != tseg) {
                    pending[keep++] = l;
                    continue;
                }
                int s_new = (int)P.lmk_order.size();
                P.lmk_order.push_back(l);
                P.lmk_first_slot[(size_t)s_new] = t * kTile + used;
                P.lmk_count[(size_t)s_new] = c;
                for (int q = 0; q < c; ++q) {
                    P.slot_obs[(size_t)(t * kTile + used + q)] = lobs[(size_t)(lptr[l] + q)];
                    P.meta[(size_t)(t * kTile + used + q)] = meta_pack(0, (uint32_t)ll);
                    scam[(size_t)(t * kTile + used + q)] = lcam[(size_t)(lptr[l] + q)];
                }
                used += c;
                ++ll;
            }
            pending.resize(keep);
            ++t;
        }
        P.lmk_store.resize((size_t)nl);
        for (int s = 0; s < nl; ++s) P.lmk_store[(size_t)P.lmk_order[s]] = s;
    }
    const int64_t tiles = (int64_t)P.tile_lmk_base.size();
    P.n_tiles = tiles;
    auto per_chunk = [&](int target) {
        return (int)std::min<int64_t>(4096, std::max<int64_t>(1, (tiles + target - 1) / target));
    };
    if (max_tiles > 0) shares = 0;
    else if (target_chunks > 0) P.max_tiles = per_chunk(target_chunks);
    // Every iteration of a batch runs the multidirectional product of those problems only
    // that fail the tau-test, and lasts as long as one chunk: with many problems the chunks
    // are made shorter, so that the few that run still fill the device.  24 ring problems of
    // 50 to 200 cameras (101,342 tiles, FP32, N = 16): 50 tiles per chunk 129 us per product,
    // 8 tiles 50 us.  Solves of such problems with 1 / 2 / 4 / 8 times as many chunks as can be
    // resident, ms: 3 problems 10.3 / 10.4 / 10.4 / 10.7, 5 12.6 / 12.4 / 12.5 / 12.7, 8 16.4 /
    // 15.9 / 15.8 / 16.3, 12 20.5 / 19.2 / 18.8 / 18.9, 16 24.3 / 22.5 / 21.6 / 21.5, 24 34.6 /
    // 30.4 / 28.7 / 28.0 (FP64, N = 4 and 45 to 90 cameras the same way): a third of the problems.
    if (cam_seg) {
        int problems = 1;
        for (int c = 1; c < np; ++c) problems += cam_seg[c] != cam_seg[c - 1];
        target_multi *= std::min(8, std::max(1, problems / 3));
    }
    if (max_tiles <= 0 && max_tiles_multi <= 0 && target_multi > 0) P.max_tiles_multi = per_chunk(target_multi);
    make_chunks(P, scam, max_slots, P.max_tiles, shares, P);
    // camera-major observations, each camera's in slot order: the work-groups of the cameras
    // that share a stretch of tiles read it at about the same time
    P.cam_obs_ptr.assign((size_t)np + 1, 0);
    for (int64_t o = 0; o < m; ++o) P.cam_obs_ptr[(size_t)cam[o] + 1]++;
    for (int k = 0; k < np; ++k) P.cam_obs_ptr[(size_t)k + 1] += P.cam_obs_ptr[(size_t)k];
    P.cam_blk.assign((size_t)np + 1, 0);
    for (int c = 0; c < np; ++c) {
        const int64_t k = P.cam_obs_ptr[(size_t)c + 1] - P.cam_obs_ptr[(size_t)c];
        const int nb = (int)((k + kCamObs - 1) / kCamObs);
        P.cam_blk[(size_t)c + 1] = P.cam_blk[(size_t)c] + nb;
        P.blk_cam.insert(P.blk_cam.end(), (size_t)nb, c);
    }
    P.cam_obs.resize((size_t)m);
    std::vector<int64_t> first_slot(P.blk_cam.size());
    {
        std::vector<int64_t> fill(P.cam_obs_ptr.begin(), P.cam_obs_ptr.end() - 1);
        for (int ch = 0; ch < P.n_chunks; ++ch) {
            for (int64_t sl = (int64_t)P.chunk_tile[(size_t)ch] * kTile; sl < (int64_t)P.chunk_tile[(size_t)ch + 1] * kTile; ++sl) {
                const int64_t o = P.slot_obs[(size_t)sl];
                if (o < 0) continue;
                const int c = scam[(size_t)sl];
                const int64_t at = fill[(size_t)c]++;
                P.cam_obs[(size_t)at] = o;
                const int64_t k = at - P.cam_obs_ptr[(size_t)c];
                if (k % kCamObs == 0) first_slot[(size_t)(P.cam_blk[(size_t)c] + k / kCamObs)] = sl;
            }
        }
    }
    P.blk_order.resize(P.blk_cam.size());
    for (size_t b = 0; b < P.blk_order.size(); ++b) P.blk_order[b] = (int32_t)b;
    std::sort(P.blk_order.begin(), P.blk_order.end(), [&](int32_t x, int32_t y) {
        const int64_t fx = first_slot[(size_t)x], fy = first_slot[(size_t)y];
        return fx < fy || (fx == fy && x < y);
    });
    return BA_OK;
}

// Number of other cameras that share at least one landmark with each camera
// (the covisibility degree, an input feature of the learned preconditioner).
void covisibility_degree(const HostPlan &P, std::vector<int32_t> &deg) {
    const int np = P.np;
    deg.assign((size_t)np, 0);
    // landmark -> its observing cameras, from the tile layout (landmarks are contiguous)
    std::vector<int64_t> lptr((size_t)P.nl + 1, 0);
    for (int s = 0; s < P.nl; ++s) lptr[(size_t)s + 1] = lptr[(size_t)s] + P.lmk_count[(size_t)s];
    std::vector<int32_t> lcam((size_t)lptr[(size_t)P.nl]);
    for (int s = 0; s < P.nl; ++s)
        for (int q = 0; q < P.lmk_count[(size_t)s]; ++q)
            lcam[(size_t)(lptr[(size_t)s] + q)] = P.obs_cam[(size_t)P.slot_obs[(size_t)(P.lmk_first_slot[(size_t)s] + q)]];
    std::vector<int32_t> stamp((size_t)np, -1);
    // camera -> landmarks via the observation CSR
    std::vector<int32_t> obs_store((size_t)P.m);
    for (int s = 0; s < P.nl; ++s)
        for (int q = 0; q < P.lmk_count[(size_t)s]; ++q)
            obs_store[(size_t)P.slot_obs[(size_t)(P.lmk_first_slot[(size_t)s] + q)]] = s;
    for (int c = 0; c < np; ++c) {
        int cnt = 0;
        stamp[(size_t)c] = c;
        for (int64_t q = P.cam_obs_ptr[(size_t)c]; q < P.cam_obs_ptr[(size_t)c + 1]; ++q) {
            const int s = obs_store[(size_t)P.cam_obs[(size_t)q]];
            for (int64_t e = lptr[(size_t)s]; e < lptr[(size_t)s + 1]; ++e) {
                const int c2 = lcam[(size_t)e];
                if (stamp[(size_t)c2] != c) {
                    stamp[(size_t)c2] = c;
                    ++cnt;
                }
            }
        }
        deg[(size_t)c] = cnt;
    }
}

void build_multi_pairs(const HostPlan &P, int N, HostMultiPlan &M, const int32_t *group_in) {
    M = HostMultiPlan();
    M.N = N;
    const int np = P.np;
    std::vector<int32_t> group((size_t)np);
    if (group_in) group.assign(group_in, group_in + np);
    else partition_groups(np, N, group.data());
    const int64_t T = P.n_tiles;
    M.mmeta.assign((size_t)T * kTile, kPad);
    M.slot_cam.assign((size_t)T * kTile, 0);
    M.pair_ll.assign((size_t)T * kTile, 0xFF);
    M.slot_ooff.assign((size_t)T * kTile, 0);
    M.tile_oidx.assign((size_t)T + 1, 0);
    M.pair_grp.assign((size_t)T * kTile, -1);
    // per tile: landmark pairs (landmark, subset) in order of first appearance.  The cameras
    // come from the chunk's list by chunk slot, which stays in cache (the caller's order of
    // the observations may be any).
    for (int ch = 0; ch < P.n_chunks; ++ch) {
        const int32_t *cams = P.part_cam.data() + P.chunk_part[(size_t)ch];
        for (int64_t t = P.chunk_tile[(size_t)ch]; t < P.chunk_tile[(size_t)ch + 1]; ++t) {
            const uint32_t *meta = P.meta.data() + t * kTile;
            uint32_t *mmeta = M.mmeta.data() + t * kTile;
            int32_t *slot_cam = M.slot_cam.data() + t * kTile, *pair_grp = M.pair_grp.data() + t * kTile;
            uint8_t *pair_ll = M.pair_ll.data() + t * kTile;
            int npairs = 0, rows = 0, q = 0;
            while (q < kTile && meta[q] != kPad) {
                const uint32_t ll = meta[q] >> 16;
                const int base = npairs, q0 = q;
                for (; q < kTile && meta[q] != kPad && meta[q] >> 16 == ll; ++q) {
                    const int c = cams[meta[q] & 0xFFFFu], g = group[(size_t)c];
                    int found = npairs - 1;
                    while (found >= base && pair_grp[found] != g) --found;
                    if (found < base) {
                        found = npairs++;
                        pair_grp[found] = g;
                        pair_ll[found] = (uint8_t)ll;
                    }
                    slot_cam[q] = c;
                    mmeta[q] = (uint32_t)found | ((uint32_t)base << 8);
                }
                const int cnt = npairs - base;
                for (int a = q0; a < q; ++a) mmeta[a] |= (uint32_t)cnt << 16;
                rows += cnt * (q - q0);
            }
            M.out_rows += rows;
            M.tile_rows = std::max(M.tile_rows, rows);
        }
    }
}

// The out-pairs (camera * N + subset) of tile t in slot order, repeats included, to `keys`
// (room for kTile * kTile); returns their number.
static int tile_outputs(const HostPlan &P, const HostMultiPlan &M, int64_t t, int64_t *keys) {
    const uint32_t *mmeta = M.mmeta.data() + t * kTile;
    int n = 0;
    for (int q = 0; q < kTile && mmeta[q] != kPad; ++q) {
        const int base = (mmeta[q] >> 8) & 0xFF, cnt = (mmeta[q] >> 16) & 0xFF;
        const int64_t k0 = (int64_t)M.slot_cam[(size_t)(t * kTile + q)] * M.N;
        for (int j = 0; j < cnt; ++j) keys[n++] = k0 + M.pair_grp[(size_t)(t * kTile + base + j)];
    }
    return n;
}

int multi_tile_outputs(const HostPlan &P, const HostMultiPlan &M) {
    int most = 0;
    std::vector<int64_t> keys((size_t)kTile * kTile);
    std::vector<int32_t> seen((size_t)P.np * M.N, -1);   // last tile that held the out-pair
    for (int64_t t = 0; t < P.n_tiles; ++t) {
        const int n = tile_outputs(P, M, t, keys.data());
        int distinct = 0;
        for (int i = 0; i < n; ++i) {
            distinct += seen[(size_t)keys[(size_t)i]] != t;
            seen[(size_t)keys[(size_t)i]] = (int32_t)t;
        }
        most = std::max(most, distinct);
    }
    return most;
}

ba_status build_multi_plan(const HostPlan &P, int N, int max_out, HostMultiPlan &M, std::string &err,
                           const int32_t *group_in) {
    build_multi_pairs(P, N, M, group_in);
    return build_multi_chunks(P, max_out, M, err);
}

ba_status build_multi_chunks(const HostPlan &P, int max_out, HostMultiPlan &M, std::string &err) {
    const int np = P.np, N = M.N;
    const int64_t T = P.n_tiles;
    // chunks over out-pairs (camera, subset), numbered within a chunk tile by tile, a tile's in
    // (camera, subset) order: the order in which the chunk's rows are written out, close to that
    // of their places (numbered as the slots name them, products of small subsets took 0.5 to 4 %
    // longer: 120 cameras, N = 29, BF16 36.4 -> 38.0 us)
    struct Seen {
        int32_t tile, chunk, local;   // the last tile and chunk that held it, its number there
    };
    std::vector<Seen> seen((size_t)np * N, Seen{-1, -1, 0});
    std::vector<int64_t> keys((size_t)kTile * kTile);
    std::vector<int64_t> part_key;                    // partial row -> camera * N + subset
    int chunk = -1, outs = 0, ntiles_in = 0;
    M.max_out = 0;
    M.oidx.resize((size_t)M.out_rows);
    int64_t at = 0;                                   // next entry of oidx
    for (int64_t t = 0; t < T; ++t) {
        const int n = tile_outputs(P, M, t, keys.data());
        int distinct = 0, fresh = 0;   // out-pairs of the tile, and those new to the chunk
        for (int i = 0; i < n; ++i) {
            Seen &e = seen[(size_t)keys[(size_t)i]];
            if (e.tile == t) continue;
            e.tile = (int32_t)t;
            ++distinct;
            fresh += e.chunk != chunk;
        }
        max_out = std::max(max_out, distinct);
        if (chunk < 0 || outs + fresh > max_out || ntiles_in >= P.max_tiles_multi ||
            P.tile_seg[(size_t)t] != M.chunk_seg.back()) {
            ++chunk;
            outs = 0;
            ntiles_in = 0;
            M.chunk_tile.push_back((int32_t)t);
            M.chunk_part.push_back((int32_t)part_key.size());
            M.chunk_seg.push_back(P.tile_seg[(size_t)t]);
        }
        M.tile_oidx[(size_t)t] = (uint32_t)at;
        const size_t first_new = part_key.size();
        for (int i = 0; i < n; ++i) {
            Seen &e = seen[(size_t)keys[(size_t)i]];
            if (e.chunk == chunk) continue;
            e.chunk = chunk;
            part_key.push_back(keys[(size_t)i]);
        }
        std::sort(part_key.begin() + (int64_t)first_new, part_key.end());
        for (size_t k = first_new; k < part_key.size(); ++k) seen[(size_t)part_key[k]].local = outs++;
        for (int i = 0; i < n; ++i) M.oidx[(size_t)at++] = (uint16_t)seen[(size_t)keys[(size_t)i]].local;
        M.max_out = std::max(M.max_out, outs);
        int off = 0;
        for (int q = 0; q < kTile && M.mmeta[(size_t)(t * kTile + q)] != kPad; ++q) {
            M.slot_ooff[(size_t)(t * kTile + q)] = (uint16_t)off;
            off += (M.mmeta[(size_t)(t * kTile + q)] >> 16) & 0xFF;
        }
        ++ntiles_in;
    }
    M.tile_oidx[(size_t)T] = (uint32_t)M.oidx.size();
    M.n_chunks = chunk + 1;
    M.chunk_tile.push_back((int32_t)T);
    M.chunk_part.push_back((int32_t)part_key.size());
    M.n_part = (int64_t)part_key.size();
    if (M.max_out > 65535) {
        err = "multidirectional product: too many (camera, subset) pairs in one tile";
        return BA_ERR_UNSUPPORTED;
    }
    // (camera, subset)-major CSR over partial rows
    const int64_t K = (int64_t)np * N;
    M.cg_ptr.assign((size_t)K + 1, 0);
    for (int64_t k : part_key) M.cg_ptr[(size_t)k + 1]++;
    for (int64_t k = 0; k < K; ++k) M.cg_ptr[(size_t)k + 1] += M.cg_ptr[(size_t)k];
    M.cg_idx.resize(part_key.size());
    std::vector<int32_t> fill(M.cg_ptr.begin(), M.cg_ptr.end() - 1);
    for (size_t i = 0; i < part_key.size(); ++i) M.cg_idx[(size_t)fill[(size_t)part_key[i]]++] = (int32_t)i;
    M.part_dst.resize(part_key.size());
    for (size_t j = 0; j < part_key.size(); ++j) M.part_dst[(size_t)M.cg_idx[j]] = (int32_t)j;
    return BA_OK;
}

}  // namespace ba
