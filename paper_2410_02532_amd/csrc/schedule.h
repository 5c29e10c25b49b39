// schedule.h -- the automatic schedule of an instance, by shape: the four-step
// split (log2 of the column length, 0 = the default split of make_plan) and
// whether fixed-step passes run resident (one workgroup holds the instance).
// The entries are chosen by timing the candidate schedules on the device
// (paper_2410_02532_amd/tune.py, which writes schedule_table.inc); the lookup
// itself is a plain table, so results do not depend on timings taken at run
// time. The batch entries apply to the
// instances of a handle whose fields fill the chip (at least kBatchPoints field
// samples in all, e.g. 2^9 instances of 2^10 points with three waves), the
// others ("alone", one instance or a few) to the rest: a handle that small is
// bound by the serial time of one tile, a full one by throughput. Handles that run the
// lone and team kernels (kLoneMax below) take lone_split instead; the alone entries
// serve what is left of them (shapes below 2^10 points, more instances than kLoneMax or
// mixed field counts). (A resident
// instance runs on one CU: in a batch it nearly always wins; alone only where
// one CU's pass beats two dependent launches per z-step, e.g. the small FP64 and
// two-wave shapes.)
#pragma once

namespace opo {

constexpr long long kBatchPoints = 1LL << 20;

struct Schedule {
    int col_log2;   // 0 = default split
    int resident;   // 1 = resident passes (shapes resident_pass serves only)
};

struct ScheduleEntry {
    int f64;        // precision: 0 FP32, 1 FP64
    int nf;         // coupled waves
    int log2nt;
    int batched;    // 0 alone (a handle below kBatchPoints), 1 in a batch
    Schedule s;
};

static const ScheduleEntry kScheduleTable[] = {
#include "schedule_table.inc"
};

inline Schedule schedule_lookup(bool f64, int nf, int log2nt, bool batched)
{
    for (const ScheduleEntry &e : kScheduleTable)
        if (e.f64 == (f64 ? 1 : 0) && e.nf == nf && e.log2nt == log2nt && e.batched == (batched ? 1 : 0))
            return e.s;
    return Schedule{0, 0};
}

// Handles that do not fill the chip, of at most kLoneMax instances of 2^10 points or more
// and one field count, run the lone and team kernels: column splits (log2 n2, 0 = default)
// by the time of one instance alone. Columns of 2^5 up to 2^14 points serve the team
// kernels; above, the default's of 2^6 are the fastest (2^16, us per z-step, FP32: 11.5
// against 13.3 with 2^5 and 15.9 with 2^7; FP64 13.8, 14.6, 17.4).
constexpr int kLoneMinLog2 = 10;
constexpr int kLoneMax = 48;   // instances: their descriptors are kernel arguments

inline int lone_split(int log2nt) { return log2nt <= 14 ? 5 : 0; }

// Two-pass instances of an FP64 batch whose launches inside a pass run mid_pass: the splits
// by its times (batches of 2^22 points, us per z-step; the table's entries are by
// mixed_pass's). Columns of 2^6 instead of 2^4: three waves 2^13 172 -> 169, 2^15 176 -> 166,
// 2^16 184 (columns of 2^5, the rows' limit) -> 180; two waves 2^12 147 -> 111, 2^16 124 ->
// 121. Returns the table's split where that stays the better one. Not for batches that run
// other kernels (two 2^13 with two 2^18, which do not share one: 84 with the table's splits,
// 90 with these).
inline int batch_split(int nf, int log2nt, int table)
{
    if (nf == 3) return log2nt == 13 || log2nt == 15 || log2nt == 16 ? 6 : table;
    return log2nt == 12 || log2nt == 16 ? 6 : table;
}

// FP32 shapes that mid_pass runs faster than mixed_pass (us a z-step, mixed_pass / mid_pass,
// batches of 2^20 .. 2^23 points): columns of 2^6 and more, or rows of 2^10 and more, always
// (0.80 to 1.01 of the time). Shorter ones are stages of radix 2 over 64-byte pieces of
// rows: three waves gain but for 2^9 points (columns of 2^4, rows of 2^5: 139 / 159, 259 /
// 306; columns and rows of 2^5 287 / 257), two waves only at 2^11 and 2^12 points (columns
// of 2^5, rows of 2^6 221 / 181; but 2^4 x 2^5 121 / 141, 2^5 x 2^5 812 / 858, 2^5 x 2^8 182
// / 193, 2^4 x 2^9 97 / 113, 2^5 x 2^9 102 / 113). For batches of one shape: in a mix of
// shapes mixed_pass is the slower again (2^9 and 2^10 points, a quarter and three quarters of
// 2^9: three waves 123 / 96 and 162 / 117, two 96 / 89 and 130 / 111, half of each 97 / 100).
inline bool mid_faster_f32(int nf, int log2n2, int log2n1)
{
    if (log2n2 >= 6 || log2n1 >= 10) return true;
    const int log2nt = log2n2 + log2n1;
    return nf == 3 ? log2nt > 9 : log2nt == 11 || log2nt == 12;
}

} // namespace opo
