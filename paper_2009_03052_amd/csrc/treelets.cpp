// Host-side treelet algebra of libscc: rooted shapes, canonical decompositions,
// unrooted shape ids and the per-k lookup tables used by the kernels.
//
// A rooted tree is its DFS bitstring (Sec. 3.2): '1' for an edge taken away
// from the root, '0' for the way back, children visited in descending
// lexicographic order of their words "1 s 0". Shapes of one size are ranked
// by ascending bitstring. The canonical decomposition takes the first child
// subtree as T'' and the rest as T' (the merge is 1, s_T'', 0, s_T'); beta_T
// is the number of children equal to that first child.
#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <memory>
#include <mutex>
#include <vector>

#include "scc_common.hpp"

namespace {

struct Word {          // a child word "1 s 0" or a shape string, MSB first
    uint32_t bits;
    int len;
};

// lexicographic comparison of two bitstrings of possibly different length;
// child words are primitive balanced strings, so neither is a prefix of the other
bool word_less(const Word &a, const Word &b)
{
    uint64_t x = a.len ? (uint64_t)a.bits << (64 - a.len) : 0;
    uint64_t y = b.len ? (uint64_t)b.bits << (64 - b.len) : 0;
    if (x != y) return x < y;
    return a.len < b.len;
}

Word concat(const Word &a, const Word &b)
{
    return Word{(a.bits << b.len) | b.bits, a.len + b.len};
}

HostShapes g_shapes;
int g_unr_n[SCC_KMAX + 1];
int g_unr_of[SCC_KMAX + 1][SCC_MAXSH];
int g_unr_min[SCC_KMAX + 1][SCC_MAXSH];
std::once_flag g_once;

int rank_of(int h, uint32_t bits)
{
    const uint32_t *b = g_shapes.bits[h];
    int n = g_shapes.r[h];
    const uint32_t *p = std::lower_bound(b, b + n, bits);
    return (p != b + n && *p == bits) ? (int)(p - b) : -1;
}

// Canonical string of the tree hanging at v (entered from p) over adjacency masks.
Word canon(const uint32_t *adj, int v, int p)
{
    Word kids[SCC_KMAX + 8];
    int nk = 0;
    for (uint32_t m = adj[v]; m; m &= m - 1) {
        int w = __builtin_ctz(m);
        if (w == p) continue;
        Word in = canon(adj, w, v);
        kids[nk++] = Word{(1u << (in.len + 1)) | (in.bits << 1), in.len + 2};
    }
    std::sort(kids, kids + nk, [](const Word &a, const Word &b) { return word_less(b, a); });
    Word s{0, 0};
    for (int i = 0; i < nk; i++) s = concat(s, kids[i]);
    return s;
}

// adjacency masks of the rooted tree with the given string (node 0 = root)
int parse(uint32_t bits, int len, uint32_t *adj)
{
    int stack[16], sp = 0, nn = 1;
    adj[0] = 0;
    stack[sp++] = 0;
    for (int i = len - 1; i >= 0; i--) {
        if (bits >> i & 1u) {
            int x = nn++;
            adj[x] = 0;
            int p = stack[sp - 1];
            adj[p] |= 1u << x;
            adj[x] |= 1u << p;
            stack[sp++] = x;
        } else {
            sp--;
        }
    }
    return nn;
}

void init_shapes()
{
    // words[s]: all child words of subtrees with s nodes, i.e. "1 s_T 0" for |T| = s
    std::vector<Word> words[SCC_KMAX + 1];
    g_shapes.r[1] = 1;
    g_shapes.bits[1][0] = 0;
    words[1].push_back(Word{0b10, 2});
    for (int h = 2; h <= SCC_KMAX; h++) {
        // children multisets with sizes summing to h-1, in non-increasing word order
        std::vector<uint32_t> found;
        std::vector<Word> cur;
        std::function<void(int, bool, Word)> rec = [&](int remaining, bool bounded, Word maxw) {
            if (remaining == 0) {
                Word s{0, 0};
                for (const Word &w : cur) s = concat(s, w);
                found.push_back(s.bits);
                return;
            }
            for (int s = 1; s <= remaining; s++)
                for (const Word &w : words[s]) {
                    if (bounded && word_less(maxw, w)) continue;
                    cur.push_back(w);
                    rec(remaining - s, true, w);
                    cur.pop_back();
                }
        };
        rec(h - 1, false, Word{0, 0});
        std::sort(found.begin(), found.end());
        found.erase(std::unique(found.begin(), found.end()), found.end());
        g_shapes.r[h] = (int)found.size();
        for (size_t i = 0; i < found.size(); i++) {
            g_shapes.bits[h][i] = found[i];
            words[h].push_back(Word{(1u << (2 * h - 1)) | (found[i] << 1), 2 * h});
        }
    }
    // unrooted classes: minimum rooted rank over all rootings, numbered ascending
    for (int h = 1; h <= SCC_KMAX; h++) {
        int minr[SCC_MAXSH];
        for (int q = 0; q < g_shapes.r[h]; q++) {
            uint32_t adj[16];
            int nn = parse(g_shapes.bits[h][q], 2 * (h - 1), adj);
            int best = SCC_MAXSH;
            for (int x = 0; x < nn; x++) best = std::min(best, rank_of(h, canon(adj, x, -1).bits));
            minr[q] = best;
        }
        std::vector<int> mins(minr, minr + g_shapes.r[h]);
        std::sort(mins.begin(), mins.end());
        mins.erase(std::unique(mins.begin(), mins.end()), mins.end());
        g_unr_n[h] = (int)mins.size();
        for (size_t j = 0; j < mins.size(); j++) g_unr_min[h][j] = mins[j];
        for (int q = 0; q < g_shapes.r[h]; q++)
            g_unr_of[h][q] = (int)(std::lower_bound(mins.begin(), mins.end(), minr[q]) - mins.begin());
    }
}

int binom(int n, int r)
{
    if (r < 0 || r > n) return 0;
    long v = 1;
    for (int i = 1; i <= r; i++) v = v * (n - r + i) / i;
    return (int)v;
}

}  // namespace

const HostShapes &host_shapes()
{
    std::call_once(g_once, init_shapes);
    return g_shapes;
}

int unrooted_count(int k)
{
    host_shapes();
    return g_unr_n[k];
}

int tree_unrooted_id(int k, const uint32_t *adjmask)
{
    host_shapes();
    int best = SCC_MAXSH;
    for (int x = 0; x < k; x++) best = std::min(best, rank_of(k, canon(adjmask, x, -1).bits));
    for (int j = 0; j < g_unr_n[k]; j++)
        if (g_unr_min[k][j] == best) return j;
    return -1;
}

static void build_dense(int k, DevLut *L);
static void build_draw(int k, DevLut *L);

void build_lut(int k, DevLut *L)
{
    const HostShapes &S = host_shapes();
    memset(L, 0, sizeof *L);
    L->k = k;
    L->off[1] = 0;
    for (int h = 1; h <= k; h++) {
        L->r[h] = S.r[h];
        L->bk[h] = binom(k, h);
        L->bk1[h] = binom(k - 1, h);
        L->W[h] = S.r[h] * binom(k - 1, h - 1);
        L->WS[h] = S.r[h] * binom(k - 1, h);
        L->off[h + 1] = L->off[h] + S.r[h] * binom(k, h);
    }
    L->nkeys = L->off[k + 1];
    L->xoff[1] = 0;
    L->soff[1] = 0;
    for (int h = 1; h <= k; h++) {
        L->xoff[h + 1] = L->xoff[h] + L->W[h];
        L->soff[h + 1] = L->soff[h] + L->WS[h];
    }
    for (int h = 2; h <= k; h++)
        for (int q = 0; q < S.r[h]; q++) {
            uint32_t s = S.bits[h][q];
            int len = 2 * (h - 1);
            // first child word: scan to the first return to depth 0
            int depth = 0, wl = 0;
            for (int i = len - 1; i >= 0; i--) {
                depth += (s >> i & 1u) ? 1 : -1;
                if (depth == 0) { wl = len - i; break; }
            }
            uint32_t first = s >> (len - wl);
            uint32_t rest = s & ((wl == len) ? 0u : ((1u << (len - wl)) - 1u));
            int hpp = wl / 2, hp = h - hpp;
            uint32_t inner = (first >> 1) & ((1u << (wl - 2)) - 1u);
            // beta: children equal to the first word
            int beta = 0;
            depth = 0;
            int start = len;
            for (int i = len - 1; i >= 0; i--) {
                depth += (s >> i & 1u) ? 1 : -1;
                if (depth == 0) {
                    int l = start - i;
                    uint32_t w = (s >> i) & ((1u << l) - 1u);
                    if (l == wl && w == first) beta++;
                    start = i;
                }
            }
            L->dec_hp[h][q] = (uint8_t)hp;
            L->dec_a[h][q] = (uint8_t)rank_of(hp, rest);
            L->dec_b[h][q] = (uint8_t)rank_of(hpp, inner);
            L->dec_beta[h][q] = (uint8_t)beta;
        }
    L->num_unr = g_unr_n[k];
    for (int q = 0; q < S.r[k]; q++) L->unr_of[q] = (uint8_t)g_unr_of[k][q];
    // designated (balanced) rootings and their orbits
    uint32_t star = 0;
    for (int i = 0; i < k - 1; i++) star = (star << 2) | 2u;
    L->star_unr = k >= 2 ? g_unr_of[k][rank_of(k, star)] : 0;
    for (int j = 0; j < 32; j++) { L->bal_rank[j] = -1; L->bal_orbit[j] = 0; }
    for (int q = 0; k >= 4 && q < S.r[k]; q++) {
        const int hpp = k - L->dec_hp[k][q];
        if (hpp < 2 || hpp > k - 2) continue;
        int8_t &b = L->bal_rank[g_unr_of[k][q]];
        if (b < 0 || q < b) b = (int8_t)q;
    }
    for (int j = 0; j < L->num_unr; j++) {
        if (L->bal_rank[j] < 0) continue;
        L->designated[L->bal_rank[j]] = 1;
        uint32_t adj[16];
        const int nn = parse(S.bits[k][L->bal_rank[j]], 2 * (k - 1), adj);
        for (int x = 0; x < nn; x++) L->bal_orbit[j] += rank_of(k, canon(adj, x, -1).bits) == L->bal_rank[j];
    }
    int cnt[SCC_KMAX + 1] = {0};
    for (uint32_t m = 0; m < (1u << (k - 1)); m++) {
        int p = __builtin_popcount(m);
        L->colex_s[m] = (uint8_t)cnt[p];
        L->mask_s[p][cnt[p]++] = (uint8_t)m;
    }
    int cntk[SCC_KMAX + 2] = {0};
    for (uint32_t m = 0; m < (1u << k); m++) {
        int p = __builtin_popcount(m);
        L->colex_k[m] = (uint8_t)cntk[p];
        L->mask_k[p][cntk[p]++] = (uint8_t)m;
    }
    int nt = 0;
    for (int h = 2; h <= k; h++)
        for (int hp = 1; hp < h; hp++) {
            L->term_base[h][hp] = (uint16_t)nt;
            int nd = binom(k - 1, h - 1);
            for (int dc = 0; dc < nd; dc++) {
                uint32_t D = L->mask_s[h - 1][dc];
                for (uint32_t sub = 0; sub < (1u << (k - 1)); sub++) {
                    if ((sub & ~D) || __builtin_popcount(sub) != hp - 1) continue;
                    L->term_x[nt] = L->colex_s[sub];
                    L->term_s[nt] = L->colex_s[D ^ sub];
                    nt++;
                }
            }
        }
    for (int i = 0; i < nt; i++) L->term_xs[i] = (uint16_t)(L->term_x[i] | (L->term_s[i] << 8));
    // per-output descriptors and keys of every level
    uint32_t no = 0;
    for (int h = 2; h <= k; h++) {
        L->out_off[h] = no;
        const int nD = L->bk1[h - 1];
        for (int o = 0; o < L->W[h]; o++, no++) {
            const int t = o / nD, dc = o - t * nD;
            const int hp = L->dec_hp[h][t], hpp = h - hp;
            const uint64_t xb = (uint64_t)(L->xoff[hp] + L->dec_a[h][t] * L->bk1[hp - 1]);
            const uint64_t sb = (uint64_t)(L->soff[hpp] + L->dec_b[h][t] * L->bk1[hpp]);
            const uint64_t nsplit = (uint64_t)binom(h - 1, hp - 1);
            const uint64_t tb = L->term_base[h][hp] + (uint64_t)dc * nsplit;
            const uint64_t desig = (h == k && L->designated[t]) ? 1u : 0u;
            L->out[no] = xb | (sb << 16) | (tb << 32) | (nsplit << 48) | ((uint64_t)L->dec_beta[h][t] << 56) | (desig << 63);
            const uint32_t D = L->mask_s[h - 1][dc];
            for (int c = 0; c < k; c++) {
                const uint32_t C = expand_in(D, c) | (1u << c);
                L->out_key[c][no] = (uint16_t)(L->off[h] + t * L->bk[h] + L->colex_k[C]);
            }
        }
    }
    build_dense(k, L);
    build_draw(k, L);
}

// Order of the m-subsets of [n] in which consecutive ones differ by exchanging one
// element (the revolving-door order: the subsets without n, then those with it in
// reverse order of the rest).
static void revolving_door(int n, int m, std::vector<uint32_t> &out)
{
    out.clear();
    if (m < 0 || m > n) return;
    if (m == 0 || m == n) { out.push_back((1u << m) - 1u); return; }
    std::vector<uint32_t> with;
    revolving_door(n - 1, m, out);
    revolving_door(n - 1, m - 1, with);
    for (size_t i = with.size(); i-- > 0;) out.push_back(with[i] | 1u << (n - 1));
}

// Orders of the colour sets whose sets without a given colour lie in fewer 128-byte lines
// of a record than the revolving-door order's, found by exchanging, moving and reversing
// sets (simulated annealing, the mean over the colours as its cost): k = 7 level 4 3.67
// lines a neighbour for 4.17 and level 5 4.75 for 5.17, k = 8 level 4 6.57 for 7.43 and
// level 5 11.43 for 12.57. The search found none for level 6 of k = 7 or 8.
static const uint8_t SETS_7_4[] = {52, 37, 44, 38, 50, 49, 42, 41, 28, 56, 25, 26, 13, 21, 14, 22, 35, 11, 19, 7};
static const uint8_t SETS_7_5[] = {45, 39, 53, 51, 57, 27, 29, 60, 58, 43, 46, 15, 30, 23, 54};
static const uint8_t SETS_8_4[] = {88, 25, 28, 56, 82, 19, 22, 50, 73, 74, 104, 76, 70, 81, 67, 84, 100, 97,
                                   112, 98, 21, 7, 13, 69, 42, 11, 26, 14, 44, 37, 38, 52, 49, 41, 35};
static const uint8_t SETS_8_5[] = {78, 106, 99, 102, 101, 116, 113, 114, 120, 108, 105, 77, 75, 71, 83, 27, 86, 90,
                                   89, 92, 30, 29, 85, 53, 45, 46, 60, 57, 58, 54, 51, 43, 39, 23, 15};
static const uint8_t *found_order(int k, int h)
{
    if (k == 7) return h == 4 ? SETS_7_4 : h == 5 ? SETS_7_5 : nullptr;
    if (k == 8) return h == 4 ? SETS_8_4 : h == 5 ? SETS_8_5 : nullptr;
    return nullptr;
}

// the dense record layout of levels 2..k and the tables that follow from it
static void build_dense(int k, DevLut *L)
{
    const uint32_t all = (1u << (k - 1)) - 1u;
    std::vector<uint32_t> ord;
    for (int h = 1; h <= k; h++) {
        // by the complements, so that runs of sets without a colour are runs of
        // complements that share it; level 2 keeps the order of S_1
        revolving_door(k - 1, k - h, ord);
        const uint8_t *found = found_order(k, h);
        for (size_t i = 0; i < ord.size(); i++) {
            const uint32_t D = found ? found[i] : all & ~ord[i];
            L->setpos[h][D] = (uint8_t)(h == 2 ? L->colex_s[D] : i);
        }
        L->plane[h] = (L->W[h] + 7) / 8 * 8;
    }
    for (int h = 2; h <= k; h++)
        for (int hp = 1; hp < h; hp++) {
            const int n = binom(k - 1, h - 1) * binom(h - 1, hp - 1);
            for (int i = L->term_base[h][hp]; i < L->term_base[h][hp] + n; i++) {
                const uint32_t D = L->mask_s[hp - 1][L->term_x[i]];
                L->xterm[i] = (uint16_t)(L->setpos[hp][D] * L->r[hp] | L->term_s[i] << 9);
            }
        }
    for (int h = 2; h <= k; h++) {
        const int nD = L->bk1[h - 1];
        for (int o = 0; o < L->W[h]; o++) {
            const int t = o / nD, dc = o - t * nD, hp = L->dec_hp[h][t];
            const int pos = L->setpos[h][L->mask_s[h - 1][dc]] * L->r[h] + t;
            const uint32_t at = L->out_off[h];
            L->xpos[at + o] = (uint16_t)pos;
            L->xord[at + pos] = (uint16_t)o;
            L->outd[at + pos] = (L->out[at + o] & ~(uint64_t)0xffffu) | (uint64_t)(L->xoff[hp] + L->dec_a[h][t]);
        }
    }
    for (int h = 2; h <= k; h++) {
        const uint64_t *d = L->outd + L->out_off[h];
        uint16_t *by = L->xsort + L->out_off[h];
        for (int i = 0; i < L->W[h]; i++) by[i] = (uint16_t)i;
        std::stable_sort(by, by + L->W[h], [d](uint16_t a, uint16_t b) { return (d[a] >> 48 & 0xffu) > (d[b] >> 48 & 0xffu); });
    }
    for (int h = 2; h < k; h++)
        for (int c = 0; c < k; c++)
            for (int q = 0; q < L->bk1[h]; q++) {
                const uint32_t C = expand_in(L->mask_s[h][q], c);
                uint64_t w = 0;
                for (int cu = 0; cu < SCC_KMAX; cu++) {
                    const uint64_t b = cu < k && (C >> cu & 1u) ? L->setpos[h][compress_out(C & ~(1u << cu), cu)] : 0xffu;
                    w |= b << (8 * cu);
                }
                L->gsel[h][c][q] = w;
            }
}

// the sampler's tables: a word per key, and the subsets of every colour set by size
static void build_draw(int k, DevLut *L)
{
    for (int h = 2; h <= k; h++)
        for (int t = 0; t < L->r[h]; t++)
            for (int ci = 0; ci < L->bk[h]; ci++) {
                const int hp = L->dec_hp[h][t], hpp = h - hp, a = L->dec_a[h][t], b = L->dec_b[h][t];
                L->kinfo[L->off[h] + t * L->bk[h] + ci] =
                    (uint64_t)L->mask_k[h][ci] | (uint64_t)h << 8 | (uint64_t)hp << 12 |
                    (uint64_t)L->dec_beta[h][t] << 16 | (uint64_t)a << 20 | (uint64_t)b << 28 |
                    (uint64_t)(L->off[hp] + a * L->bk[hp]) << 36 | (uint64_t)(L->off[hpp] + b * L->bk[hpp]) << 48;
            }
    for (int c = 0; c < k; c++) L->kinfo[c] = (uint64_t)(1u << c) | 1ull << 8;   // level 1
    int at = 0;
    for (uint32_t R = 0; R < (1u << k); R++)
        for (int m = 0; m <= __builtin_popcount(R); m++) {
            L->sub_at[R][m] = (uint16_t)at;
            for (uint32_t s = 0; s <= R; s++)
                if (!(s & ~R) && __builtin_popcount(s) == m) L->subs[at++] = (uint8_t)s;
        }
}

// ---------------------------------------------------------------------------
// errors
// ---------------------------------------------------------------------------
static thread_local char t_err[512];

scc_status set_error(scc_status st, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(t_err, sizeof t_err, fmt, ap);
    va_end(ap);
    return st;
}

extern "C" const char *scc_last_error(void) { return t_err; }
extern "C" const char *scc_version(void) { return "scc-mi355x 0.1 (gfx950)"; }
extern "C" int scc_num_unrooted(int k) { return (k >= 1 && k <= SCC_KMAX) ? unrooted_count(k) : -1; }

extern "C" int scc_balanced_rooting(int k, int j, int *orbit)
{
    if (orbit) *orbit = 0;
    if (k < 1 || k > SCC_KMAX || j < 0 || j >= unrooted_count(k)) return -1;
    std::unique_ptr<DevLut> L(new DevLut);   // ~50 KB: not on the caller's stack
    build_lut(k, L.get());
    if (orbit) *orbit = L->bal_orbit[j];
    return L->bal_rank[j];
}

extern "C" int scc_star_shape(int k)
{
    if (k < 2 || k > SCC_KMAX) return -1;
    std::unique_ptr<DevLut> L(new DevLut);
    build_lut(k, L.get());
    return L->star_unr;
}

void *DevMem::get(size_t bytes)
{
    if (bytes == 0) bytes = 256;
    if (alloc && alloc->alloc) return alloc->alloc(bytes, (void *)stream, alloc->ctx);
    void *p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) return nullptr;
    return p;
}

void DevMem::put(void *p)
{
    if (!p) return;
    if (alloc && alloc->free) alloc->free(p, (void *)stream, alloc->ctx);
    else (void)hipFree(p);
}
